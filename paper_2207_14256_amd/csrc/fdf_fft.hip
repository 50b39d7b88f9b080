// Potential grids and power spectra: Fourier stage + 3-D Stockham FFTs (gfx950).
//
// Inverse direction (grid build, sec. 2.1 "potential grids"): delta_0(k) is
// multiplied by the transfer functions and i k_a, then transformed by three
// passes, in registers with LDS between the stages:
//   X pass  : strided C2C along x, fused with the Fourier-stage multipliers;
//             one block = NB consecutive z-columns of one y row, all x;
//   Y pass  : strided C2C along y, in place;
//   Z pass  : contiguous C2R along z through a half-length complex FFT,
//             writing all slots of a cell together (packed [G^3][nslot]).
// Forward direction (P(k), sec. 4): Z pass R2C, Y pass, X pass in place (or,
// for the momentum spectrum, multiplied by i k_a and summed over the axes),
// then exact log-|k| binning of Re(A conj B) in fixed point.
//
// Half-complex intermediates keep only n_z in [0, G/2): every Nyquist mode
// of delta_0 is zero, and the spectrum bins stop below k_N, so the n_z = G/2
// plane is never needed.
//
// Stockham stage (radix R, Ns = product of earlier radices), for butterfly j:
//   v_r = in[j + r N/R] * W_{Ns R}^{r (j mod Ns)},  v = DFT_R(v),
//   out[(j/Ns) Ns R + (j mod Ns) + r Ns] = v_r.
#include <type_traits>

#include "fdf_device.h"
#include "fdf_internal.h"

namespace fdf {
namespace {

// ------------------------------------------------------------ butterflies --
template <bool INV, typename R>
__device__ __forceinline__ void bfly2(cplx<R>* v) {
  cplx<R> a = cadd(v[0], v[1]), b = csub(v[0], v[1]);
  v[0] = a; v[1] = b;
}

template <bool INV, typename R>
__device__ __forceinline__ void bfly4(cplx<R>& v0, cplx<R>& v1, cplx<R>& v2, cplx<R>& v3) {
  cplx<R> a0 = cadd(v0, v2), a1 = csub(v0, v2), a2 = cadd(v1, v3), a3 = csub(v1, v3);
  v0 = cadd(a0, a2);
  v2 = csub(a0, a2);
  if (INV) {  // X1 = a1 + i a3, X3 = a1 - i a3
    v1 = {a1.x - a3.y, a1.y + a3.x};
    v3 = {a1.x + a3.y, a1.y - a3.x};
  } else {    // X1 = a1 - i a3, X3 = a1 + i a3
    v1 = {a1.x + a3.y, a1.y - a3.x};
    v3 = {a1.x - a3.y, a1.y + a3.x};
  }
}

template <bool INV, typename R>
__device__ __forceinline__ void bfly8(cplx<R>* v) {
  const R c = (R)0.70710678118654752440084436210484903928;
  cplx<R> e0 = v[0], e1 = v[2], e2 = v[4], e3 = v[6];
  cplx<R> o0 = v[1], o1 = v[3], o2 = v[5], o3 = v[7];
  bfly4<INV>(e0, e1, e2, e3);
  bfly4<INV>(o0, o1, o2, o3);
  cplx<R> t1, t2, t3;
  if (INV) {  // W8^s = e^{+i pi s/4}
    t1 = {c * (o1.x - o1.y), c * (o1.x + o1.y)};
    t2 = {-o2.y, o2.x};
    t3 = {-c * (o3.x + o3.y), c * (o3.x - o3.y)};
  } else {    // W8^s = e^{-i pi s/4}
    t1 = {c * (o1.x + o1.y), c * (o1.y - o1.x)};
    t2 = {o2.y, -o2.x};
    t3 = {c * (o3.y - o3.x), -c * (o3.x + o3.y)};
  }
  v[0] = cadd(e0, o0); v[4] = csub(e0, o0);
  v[1] = cadd(e1, t1); v[5] = csub(e1, t1);
  v[2] = cadd(e2, t2); v[6] = csub(e2, t2);
  v[3] = cadd(e3, t3); v[7] = csub(e3, t3);
}

template <int RAD, bool INV, typename R>
__device__ __forceinline__ void bfly(cplx<R>* v) {
  if constexpr (RAD == 8) bfly8<INV>(v);
  else if constexpr (RAD == 4) bfly4<INV>(v[0], v[1], v[2], v[3]);
  else bfly2<INV>(v);
}

// ------------------------------------------------------------- LDS lines --
// NB lines of length N, transformed together by NT threads that hold their
// elements in registers: every stage works on registers and the lines pass
// through LDS only between two stages, so that the caller reads its input
// straight into the first stage's registers and takes its results out of the
// last stage's (two exchanges and four barriers for 256 = 8 8 4).  The barriers
// order LDS alone; global loads and stores stay in flight across them.
// tw is the global table e^{-2 pi i m / G}; the length-N root of unity W_N^m
// is tw[m * TWS] with TWS = G / N.  HOLD keeps a thread's twiddles in
// registers (once per block instead of once per line group).
// Element n of line b is at buf[at(n, b)] of kSize elements: rows of NB, with
// a spare row after every eight, because the first stage's results are written
// at a stride of 8 rows.  XL is for callers whose neighbouring threads hold
// neighbouring elements of one line: the row bits that pick the bank group are
// mixed with the next higher ones and the line bits with those above.
template <typename R, int N, int NB, int NT, bool INV, int TWS, bool HOLD, bool XL = false>
struct Lines {
  static constexpr int E = NB * N / NT > 8 ? NB * N / NT : 8;   // elements per thread
  static constexpr int ROW = NB * (int)sizeof(cplx<R>);
  static constexpr int Q = ROW >= 256 ? 1 : ROW <= 32 ? 8 : 256 / ROW;   // rows per sweep of the banks
  static constexpr int QSH = Q == 8 ? 3 : Q == 4 ? 2 : Q == 2 ? 1 : 0;
  static constexpr int radix(int ns) { return N / ns >= 8 ? 8 : N / ns; }
  static constexpr int per(int ns) { return (NB * (N / radix(ns)) + NT - 1) / NT; }
  static constexpr bool whole(int ns) { return (NB * (N / radix(ns))) % NT == 0; }
  // the twiddles of a stage are the same for all of a thread's butterflies
  static constexpr bool shared(int ns) { return NT % NB == 0 && (NT / NB) % ns == 0; }
  static constexpr int tw_count(int ns) { return (radix(ns) - 1) * (shared(ns) ? 1 : per(ns)); }
  static constexpr int tw_offset(int ns) {
    int o = 0;
    for (int q = radix(1); q < ns; q *= radix(q)) o += tw_count(q);
    return o;
  }

  static constexpr int kSize = XL ? N * NB : (N + N / 8) * NB;
  static __device__ __forceinline__ int at(unsigned n, unsigned b) {
    if constexpr (XL) return (n ^ ((n >> 3) & (Q - 1))) * NB + (b ^ ((n >> QSH) & (NB - 1)));
    else return (n + n / 8) * NB + b;
  }
  // at(n + dn, b), dn a constant: a fixed distance where a whole number of eights apart
  static __device__ __forceinline__ int at(unsigned n, int dn, unsigned b) {
    return !XL && dn % 8 == 0 ? at(n, b) + (dn + dn / 8) * NB : at(n + dn, b);
  }

  // Register i of a thread holds element tid / NB + dn of line tid % NB as the
  // stage that follows NS points expects it: f(dn, i), where dn is a constant
  // once the loops are unrolled, so that addresses are a scalar part and one
  // vector offset per thread.
  template <int NS, typename F> static __device__ __forceinline__ void inputs(int tid, F f) {
    static_assert(NT % NB == 0, "a thread keeps its line");
    constexpr int RAD = radix(NS);
#pragma unroll
    for (int p = 0; p < per(NS); ++p) {
      if (whole(NS) || tid + p * NT < NB * (N / RAD)) {
#pragma unroll
        for (int r = 0; r < RAD; ++r) f(p * (NT / NB) + r * (N / RAD), p * RAD + r);
      }
    }
  }
  template <typename F> static __device__ __forceinline__ void first(int tid, F f) { inputs<1>(tid, f); }
  static __device__ __forceinline__ void first(cplx<R>* v, int tid, const cplx<R>* buf) {
    first(tid, [&](int dn, int i) { v[i] = buf[at(tid / NB, dn, tid % NB)]; });
  }

  struct Twiddles {
    const cplx<R>* __restrict__ tw;
    cplx<R> w[HOLD && tw_offset(N) > 0 ? tw_offset(N) : 1];
    template <int NS> __device__ __forceinline__ void fetch(int tid) {
      if constexpr (NS < N) {
        if constexpr (NS > 1) {
          constexpr int RAD = radix(NS), O = tw_offset(NS);
#pragma unroll
          for (int p = 0; p < (shared(NS) ? 1 : per(NS)); ++p) {
            if (!whole(NS) && tid + p * NT >= NB * (N / RAD)) continue;
            const int k = ((tid + p * NT) / NB) % NS;
#pragma unroll
            for (int r = 1; r < RAD; ++r) w[O + p * (RAD - 1) + r - 1] = tw[(r * k * (N / (NS * RAD))) * TWS];
          }
        }
        fetch<NS * radix(NS)>(tid);
      }
    }
    __device__ __forceinline__ Twiddles(const cplx<R>* t, int tid) : tw(t) {
      if constexpr (HOLD) fetch<1>(tid);
    }
    template <int NS> __device__ __forceinline__ cplx<R> get(int p, int r, int k) const {
      constexpr int RAD = radix(NS), O = tw_offset(NS);
      if constexpr (HOLD) return w[O + (shared(NS) ? 0 : p) * (RAD - 1) + r - 1];
      else return tw[(r * k * (N / (NS * RAD))) * TWS];
    }
  };

  // v: the first stage's inputs; sink(dn, z) gets element tid / NB + dn of line
  // tid % NB.  Every read of buf is behind the last barrier, so that the next
  // call may follow at once.
  template <int NS = 1, typename F>
  static __device__ __forceinline__ void run(cplx<R>* v, int tid, cplx<R>* buf, const Twiddles& w, F sink) {
    constexpr int RAD = radix(NS);
#pragma unroll
    for (int p = 0; p < per(NS); ++p) {
      if (whole(NS) || tid + p * NT < NB * (N / RAD)) {
        const int b = tid % NB, j = tid / NB + p * (NT / NB);
        const int k = j % NS;
        if constexpr (NS > 1) {
#pragma unroll
          for (int r = 1; r < RAD; ++r) {
            const cplx<R> z = w.template get<NS>(p, r, k);
            v[p * RAD + r] = INV ? cmulc(v[p * RAD + r], z) : cmul(v[p * RAD + r], z);
          }
        }
        bfly<RAD, INV>(v + p * RAD);
        const int base = (j / NS) * NS * RAD + k;
#pragma unroll
        for (int r = 0; r < RAD; ++r) {
          if constexpr (NS * RAD < N) buf[NS == 1 && !XL ? at(base, b) + r * NB : at(base, r * NS, b)] = v[p * RAD + r];
          else sink(p * (NT / NB) + r * NS, v[p * RAD + r]);   // j < NS: base = j
        }
      }
    }
    if constexpr (NS * RAD < N) {
      lds_barrier();
      inputs<NS * RAD>(tid, [&](int dn, int i) { v[i] = buf[at(tid / NB, dn, tid % NB)]; });
      lds_barrier();
      run<NS * RAD>(v, tid, buf, w, sink);
    }
  }
};

// ---------------------------------------------------------- block shapes --
template <typename R, int G> struct Shape {
  static constexpr int CS = (int)sizeof(cplx<R>);
  static constexpr int NB0 = 65536 / (G * CS);
  static constexpr int NB = NB0 > 16 ? 16 : (NB0 < 1 ? 1 : NB0);     // columns per strided block
  static constexpr int NBC = NB > G / 2 ? G / 2 : NB;
  static constexpr int NTS0 = NBC * G / 16;                          // 16 elements per thread
  static constexpr int NTS = NTS0 < 64 ? 64 : NTS0;                  // threads per strided block
  static constexpr int NTX0 = NBC * G < 256 ? NBC * G : 256;          // inverse X pass: at least
  static constexpr int NTX1 = CS > 8 ? (2 * NTS > 1024 ? 1024 : 2 * NTS) : NTS;   // binary64: 8 elements
  static constexpr int NTX = NTX1 < NTX0 ? NTX0 : NTX1;
  static constexpr int NT = 256;
  static constexpr int M = G / 2;
  static constexpr int NL0 = 1024 / G;
  static constexpr int NL1 = NL0 > 16 ? 16 : (NL0 < 1 ? 1 : NL0);
  static constexpr int NL = NL1 > G ? G : NL1;                        // lines per contiguous block
};

__device__ __forceinline__ int signed_index(int i, int G) { return i < G / 2 ? i : i - G; }

// Transfer function of one slot at k^2 (times i k_a for the gradients).
enum TransferKind : int32_t { TK_ZERO, TK_PHIDOT, TK_PHI, TK_PSI, TK_PHI_PSI };
__device__ __forceinline__ int transfer_kind(int kind) {
  switch (kind) {
    case SK_DX_PSI: case SK_DY_PSI: case SK_DZ_PSI: case SK_PSI: return TK_PSI;
    case SK_DX_PHI: case SK_DY_PHI: case SK_DZ_PHI: case SK_PHI: return TK_PHI;
    case SK_PHIDOT: return TK_PHIDOT;
    case SK_PHI_PSI: return TK_PHI_PSI;
    default: return TK_ZERO;
  }
}
__device__ __forceinline__ double transfer(int tk, double k2, const Transfer& tr) {
  if (k2 == 0.0 || tk == TK_ZERO) return 0.0;
  if (tk == TK_PHIDOT) return tr.c_phidot / k2;
  const double tphi = tr.c_phi / k2;
  if (tk == TK_PHI) return tphi;
  const double tpsi = tphi * (1.0 - tr.slip_amp * exp(-sqrt(k2) / tr.slip_k));
  return tk == TK_PSI ? tpsi : tphi + tpsi;
}

// ------------------------------------------------------------------ X pass --
// The transfer function of a thread's modes is kept over the slots that share
// it (three gradient components, as a rule): its binary64 square root,
// exponential and division are the pass's longest arithmetic.  16 elements per
// thread in binary32 (8 in binary64), the modes, their transfer function and
// the twiddles in registers: two waves per SIMD, and still faster than with the
// modes read again (198 us) or the twiddles (172 us).
// 7 slots of 256^3 in binary32 (0.54 GB): 249 us with the lines in LDS through
// every stage and a transfer function per slot, 160 us.  6 slots of 512^3:
// 2.14 -> 1.21 ms.  The binary64 form: 350 -> 301 us.  Splitting the slots over
// several X-Y launch pairs, so that the second pass finds its planes in the
// memory-side cache, takes from the Y pass what the X pass loses.
template <typename R, int G>
__global__ void __launch_bounds__((Shape<R, G>::NTX)) k_xpass_inverse(GridBuildArgs a) {
  using S = Shape<R, G>;
  constexpr int NB = S::NBC, M = S::M;
  constexpr bool kHold = sizeof(R) == 4;   // binary64: registers run out
  using L = Lines<R, G, NB, S::NTX, true, 1, kHold>;
  __shared__ union { cplx<R> lines[L::kSize]; double t[G * NB]; } lds;
  cplx<R>* const buf = lds.lines;
  double* const tbuf = lds.t;
  const int nzb = M / NB, tid = threadIdx.x;
  const int iy = blockIdx.x / nzb, iz0 = (blockIdx.x % nzb) * NB;
  const cplx<R>* __restrict__ din = (const cplx<R>*)a.delta_k + (size_t)iy * M + iz0;
  cplx<R>* const scr = (cplx<R>*)a.scratch + (size_t)iy * M + iz0;
  const uint32_t at = (uint32_t)(tid / NB) * (G * M) + tid % NB;
  const size_t plane = (size_t)G * G * M;
  const typename L::Twiddles tw((const cplx<R>*)a.twiddle, tid);
  const int ny = signed_index(iy, G), nz = iz0 + tid % NB;
  cplx<R> d[kHold ? L::E : 1], v[L::E];
  double t[L::E];
  if constexpr (kHold) L::first(tid, [&](int dn, int i) { d[i] = (din + (size_t)dn * (G * M))[at]; });
  int held = -1;
#pragma unroll 1
  for (int f = 0; f < a.nfft; ++f) {
    const int kind = a.kind[f], tk = transfer_kind(kind);
    int n0 = tid / NB;
    asm volatile("" : "+v"(n0));   // the wave numbers stay in the loop: E of them would be held across it
    if (tk != held) {
      // evaluated in a loop, through the idle buffer: side by side in
      // registers, the evaluations would leave room for one wave per SIMD
#pragma unroll 2
      for (int e = tid; e < G * NB; e += S::NTX) {
        const int nx = signed_index(e / NB, G);
        tbuf[e] = transfer(tk, a.kf * a.kf * (double)(nx * nx + ny * ny + nz * nz), a.tr);
      }
      lds_barrier();
      L::first(tid, [&](int dn, int i) { t[i] = tbuf[tid + dn * NB]; });
      lds_barrier();
      held = tk;
    }
    // multiplier re + i im = T or i k_a T, without branches: re = T or 0, and
    // the gradient's wave number n_a = ax n_x + na (0 for T itself)
    const int ax = kind == SK_DX_PSI || kind == SK_DX_PHI;
    const int na = kind == SK_DY_PSI || kind == SK_DY_PHI ? ny : kind == SK_DZ_PSI || kind == SK_DZ_PHI ? nz : 0;
    const double one = kind >= SK_DX_PSI && kind <= SK_DZ_PHI ? 0.0 : 1.0;
    L::first(tid, [&](int dn, int i) {
      cplx<R> z;
      if constexpr (kHold) {
        asm("" : "+v"(d[i].x), "+v"(d[i].y));   // nor are the modes held in binary64
        z = d[i];
      }
      else z = (din + (size_t)dn * (G * M))[at];
      const double re = one * t[i], im = a.kf * (double)(ax * signed_index(n0 + dn, G) + na) * t[i];
      const double dx = (double)z.x, dy = (double)z.y;
      v[i] = {(R)(re * dx - im * dy), (R)(re * dy + im * dx)};
      if (kHold && i % 2 == 1) __builtin_amdgcn_sched_barrier(0);
    });
    cplx<R>* const out = scr + f * plane;
    L::run(v, tid, buf, tw, [&](int dn, cplx<R> z) { (out + (size_t)dn * (G * M))[at] = z; });
  }
}

// ------------------------------------------------- Y pass (either direction) --
// blocks over (field h, ix, z-column block); lines along y; in place.  7 planes
// of 256^3 in binary32 (0.94 GB): 350 -> 176 us with one LDS exchange between
// two stages instead of LDS in front of and behind every stage; what is left is
// the rate of a copy.  6 planes of 512^3 ran at that rate before (1.40 ms, 1.44).
template <typename R, int G, bool INV>
__global__ void __launch_bounds__((Shape<R, G>::NTS)) k_ypass(cplx<R>* scr, const cplx<R>* __restrict__ twiddle) {
  using S = Shape<R, G>;
  constexpr int NB = S::NBC, M = S::M;
  using L = Lines<R, G, NB, S::NTS, INV, 1, true>;
  __shared__ cplx<R> buf[L::kSize];
  const int nzb = M / NB, tid = threadIdx.x;
  const int blk = blockIdx.x;
  const int izb = blk % nzb, ix = (blk / nzb) % G, f = blk / (nzb * G);
  cplx<R>* const base = scr + (size_t)f * G * G * M + (size_t)ix * G * M + izb * NB;
  const uint32_t at = (uint32_t)(tid / NB) * M + tid % NB;
  cplx<R> v[L::E];
  L::first(tid, [&](int dn, int i) { v[i] = (base + (size_t)dn * M)[at]; });
  const typename L::Twiddles tw(twiddle, tid);
  L::run(v, tid, buf, tw, [&](int dn, cplx<R> z) { (base + (size_t)dn * M)[at] = z; });
}

// ------------------------------------------------ Z pass: C2R + slot packing --
template <int NSLOT, int OT, typename R>
__device__ __forceinline__ void store_cell(void* out, size_t cell, const R* vals);

template <> __device__ __forceinline__ void store_cell<8, GT_BF16, float>(void* out, size_t cell, const float* v) {
  uint4 w;
  w.x = f32_to_bf16_bits(v[0]) | (f32_to_bf16_bits(v[1]) << 16);
  w.y = f32_to_bf16_bits(v[2]) | (f32_to_bf16_bits(v[3]) << 16);
  w.z = f32_to_bf16_bits(v[4]) | (f32_to_bf16_bits(v[5]) << 16);
  w.w = f32_to_bf16_bits(v[6]) | (f32_to_bf16_bits(v[7]) << 16);
  ((uint4*)out)[cell] = w;
}
template <> __device__ __forceinline__ void store_cell<6, GT_BF16, float>(void* out, size_t cell, const float* v) {
  uint32_t* o = (uint32_t*)out + 3 * cell;   // 12-byte cell
  o[0] = f32_to_bf16_bits(v[0]) | (f32_to_bf16_bits(v[1]) << 16);
  o[1] = f32_to_bf16_bits(v[2]) | (f32_to_bf16_bits(v[3]) << 16);
  o[2] = f32_to_bf16_bits(v[4]) | (f32_to_bf16_bits(v[5]) << 16);
}
template <> __device__ __forceinline__ void store_cell<4, GT_BF16, float>(void* out, size_t cell, const float* v) {
  uint2 w;
  w.x = f32_to_bf16_bits(v[0]) | (f32_to_bf16_bits(v[1]) << 16);
  w.y = f32_to_bf16_bits(v[2]) | (f32_to_bf16_bits(v[3]) << 16);
  ((uint2*)out)[cell] = w;
}
template <> __device__ __forceinline__ void store_cell<4, GT_F32, float>(void* out, size_t cell, const float* v) {
  ((float4*)out)[cell] = make_float4(v[0], v[1], v[2], v[3]);
}
template <> __device__ __forceinline__ void store_cell<8, GT_F32, float>(void* out, size_t cell, const float* v) {
  ((float4*)out)[2 * cell] = make_float4(v[0], v[1], v[2], v[3]);
  ((float4*)out)[2 * cell + 1] = make_float4(v[4], v[5], v[6], v[7]);
}
template <> __device__ __forceinline__ void store_cell<4, GT_F64, double>(void* out, size_t cell, const double* v) {
  double2* o = (double2*)out + 2 * cell;
  o[0] = make_double2(v[0], v[1]);
  o[1] = make_double2(v[2], v[3]);
}
template <> __device__ __forceinline__ void store_cell<6, GT_F64, double>(void* out, size_t cell, const double* v) {
  double2* o = (double2*)out + 3 * cell;
  o[0] = make_double2(v[0], v[1]);
  o[1] = make_double2(v[2], v[3]);
  o[2] = make_double2(v[4], v[5]);
}
template <> __device__ __forceinline__ void store_cell<8, GT_F64, double>(void* out, size_t cell, const double* v) {
  double2* o = (double2*)out + 4 * cell;
  o[0] = make_double2(v[0], v[1]);
  o[1] = make_double2(v[2], v[3]);
  o[2] = make_double2(v[4], v[5]);
  o[3] = make_double2(v[6], v[7]);
}

// Half-length pre-processing of one line's pair (k, M - k), 0 < k < M / 2; the
// pair of k = 0 is made of the two elements that are their own partners, k = 0
// (whose partner X[M], a Nyquist mode, is zero) and k = M / 2.
// Z[k] = (X[k] + conj X[M-k]) + i e^{2 pi i k/G} (X[k] - conj X[M-k])
template <typename R>
__device__ __forceinline__ cplx<R> c2r_element(cplx<R> xk, cplx<R> xm, cplx<R> w) {
  cplx<R> s = {xk.x + xm.x, xk.y - xm.y};          // X[k] + conj X[M-k]
  cplx<R> d = {xk.x - xm.x, xk.y + xm.y};          // X[k] - conj X[M-k]
  cplx<R> wd = cmulc(d, w);                        // d e^{+2 pi i k/G}
  return {s.x - wd.y, s.y + wd.x};                 // s + i wd
}

// blocks over (ix, y-line block of NL lines)
template <typename R, int G, int NSLOT, int OT>
__global__ void __launch_bounds__(256) k_zpass_c2r(GridBuildArgs a) {
  using S = Shape<R, G>;
  constexpr int NL = S::NL, NT = S::NT, M = S::M, H = M / 2;
  using L = Lines<R, M, NL, NT, true, 2, true, true>;
  __shared__ cplx<R> buf[M * NL];
  __shared__ R stage[NL * G * NSLOT];
  const int nyb = G / NL, tid = threadIdx.x;
  const int ix = blockIdx.x / nyb, iy0 = (blockIdx.x % nyb) * NL;
  const cplx<R>* __restrict__ twiddle = (const cplx<R>*)a.twiddle;
  const cplx<R>* scr = (const cplx<R>*)a.scratch + ((size_t)ix * G + iy0) * M;
  const size_t plane = (size_t)G * G * M;
  const typename L::Twiddles tw(twiddle, tid);
  for (int e = tid; e < NL * G * NSLOT; e += NT) stage[e] = (R)0;
  lds_barrier();
  for (int f = 0; f < a.nfft; ++f) {
    const int slot = a.slot[f];
    for (int e = tid; e < H * NL; e += NT) {   // coalesced: consecutive threads, consecutive k
      const int line = e / H, k = e % H, m = k ? M - k : H;
      const cplx<R> xk = scr[f * plane + line * M + k], xm = scr[f * plane + line * M + m];
      buf[L::at(k, line)] = c2r_element(xk, k ? xm : cplx<R>{(R)0, (R)0}, twiddle[k]);
      buf[L::at(m, line)] = c2r_element(xm, k ? xk : xm, twiddle[m]);
    }
    lds_barrier();
    cplx<R> v[L::E];
    L::first(v, tid, buf);
    lds_barrier();
    L::run(v, tid, buf, tw, [&](int dn, cplx<R> z) {
      const int m = tid / NL + dn, line = tid % NL;
      stage[(line * G + 2 * m) * NSLOT + slot] = z.x;
      stage[(line * G + 2 * m + 1) * NSLOT + slot] = z.y;
    });
  }
  lds_barrier();
  for (int e = tid; e < NL * G; e += NT) {
    const int line = e / G, iz = e % G;
    const size_t cell = (size_t)mesh_x(ix, G) + mesh_y(iy0 + line, G) + mesh_z(iz);   // bricked layout
    store_cell<NSLOT, OT, R>(a.out, cell, &stage[e * NSLOT]);
  }
}

// ---------------------------------------------------- forward Z pass: R2C --
// blocks over (half h, ix, y-line block)
template <typename R, int G>
__global__ void __launch_bounds__(256) k_zpass_r2c(PkArgs a) {
  using S = Shape<R, G>;
  constexpr int NL = S::NL, NT = S::NT, M = S::M, H = M / 2;
  using L = Lines<R, M, NL, NT, false, 2, sizeof(R) == 4, true>;
  __shared__ cplx<R> buf[M * NL];
  const int nyb = G / NL, tid = threadIdx.x;
  const int blk = blockIdx.x;
  const int h = blk / (G * nyb);
  const int ix = (blk / nyb) % G, iy0 = (blk % nyb) * NL;
  const cplx<R>* __restrict__ twiddle = (const cplx<R>*)a.twiddle;
  const size_t row0 = ((size_t)ix * G + iy0) * M;
  const cplx<R>* src = (const cplx<R>*)(h ? a.grid_b : a.grid_a) + row0;   // reals read in pairs
  cplx<R>* dst = (cplx<R>*)a.scratch + (size_t)h * G * G * M + row0;
  for (int e = tid; e < M * NL; e += NT) buf[L::at(e % M, e / M)] = src[e];   // z[m] = x[2m] + i x[2m+1]
  const typename L::Twiddles tw(twiddle, tid);
  lds_barrier();
  cplx<R> v[L::E];
  L::first(v, tid, buf);
  lds_barrier();
  L::run(v, tid, buf, tw, [&](int dn, cplx<R> z) { buf[L::at(tid / NL + dn, tid % NL)] = z; });
  lds_barrier();
  // X[k] = (Z[k] + conj Z[M-k])/2 - (i/2) e^{-2 pi i k/G} (Z[k] - conj Z[M-k]),  Z[M] = Z[0]
  auto element = [&](cplx<R> zk, cplx<R> zm, cplx<R> w) -> cplx<R> {
    cplx<R> s = {zk.x + zm.x, zk.y - zm.y};
    cplx<R> d = {zk.x - zm.x, zk.y + zm.y};
    cplx<R> wd = cmul(d, w);                           // d e^{-2 pi i k/G}
    return {(R)0.5 * (s.x + wd.y), (R)0.5 * (s.y - wd.x)};   // s/2 - (i/2) wd
  };
  for (int e = tid; e < H * NL; e += NT) {
    const int line = e / H, k = e % H, m = k ? M - k : H;
    const cplx<R> zk = buf[L::at(k, line)], zm = buf[L::at(m, line)];
    dst[line * M + k] = element(zk, k ? zm : zk, twiddle[k]);
    dst[line * M + m] = element(zm, k ? zk : zm, twiddle[m]);
  }
}

// ------------------------- forward X pass + i k_axis, summed over the axes --
// Density spectrum (deriv_axis < 0): the x transform of each half, in place.
// Momentum spectrum: Theta = sum_a i k_a J_a(k), one axis per call, summed
// into planes 2 (and 3).
template <typename R, int G>
__global__ void __launch_bounds__((Shape<R, G>::NTS)) k_xpass_accum(PkArgs a) {
  using S = Shape<R, G>;
  constexpr int NB = S::NBC, M = S::M;
  using L = Lines<R, G, NB, S::NTS, false, 1, true>;
  __shared__ cplx<R> buf[L::kSize];
  const int nzb = M / NB, tid = threadIdx.x;
  const int h = blockIdx.x / (G * nzb);
  const int blk = blockIdx.x % (G * nzb);
  const int iy = blk / nzb, iz0 = (blk % nzb) * NB;
  const size_t plane = (size_t)G * G * M;
  cplx<R>* const src = (cplx<R>*)a.scratch + h * plane + (size_t)iy * M + iz0;
  const uint32_t at = (uint32_t)(tid / NB) * (G * M) + tid % NB;
  cplx<R> v[L::E];
  L::first(tid, [&](int dn, int i) { v[i] = (src + (size_t)dn * (G * M))[at]; });
  const typename L::Twiddles tw((const cplx<R>*)a.twiddle, tid);
  if (a.deriv_axis < 0) {   // each block owns its columns: in place is safe
    L::run(v, tid, buf, tw, [&](int dn, cplx<R> z) { (src + (size_t)dn * (G * M))[at] = z; });
    return;
  }
  cplx<R>* const acc = src + 2 * plane;
  const int ny = signed_index(iy, G);
  L::run(v, tid, buf, tw, [&](int dn, cplx<R> z) {
    const int na = a.deriv_axis == 0 ? signed_index(tid / NB + dn, G) : a.deriv_axis == 1 ? ny : iz0 + tid % NB;
    const R kn = (R)(a.kf * (double)na);
    const cplx<R> t = {-kn * z.y, kn * z.x};          // i k_axis z
    cplx<R>* const q = (acc + (size_t)dn * (G * M)) + at;
    if (a.accum_first) *q = t;
    else *q = {q->x + t.x, q->y + t.y};
  });
}

// Log binning of planes bin_plane (and bin_plane + 1), laid out [kx][ky][kz]:
// per bin the mode count, the sum of |n| and the sum of P = V Re(A conj B)
// (modes with n_z > 0 count twice).  The sums are exact integer sums, so the
// result does not depend on the order of the additions (bit for bit the same
// from run to run): |n| in units of 2^-50 and P in units of 2^(e - 61), with
// 2^e above every |P| (from a first pass), accumulated in 128 bits (a low
// word whose carry goes to a high word) with 64-bit atomics.
__device__ __forceinline__ int mode_bin(size_t gi, int G, int nbins, long* n2_out, int* nz_out) {
  const int M = G / 2;
  const int nz = (int)(gi % M), iy = (int)((gi / M) % G), ix = (int)(gi / ((size_t)M * G));
  const int nx = signed_index(ix, G), ny = signed_index(iy, G);
  const long n2 = (long)nx * nx + (long)ny * ny + (long)nz * nz;
  *n2_out = n2;
  *nz_out = nz;
  if (n2 == 0) return -1;
  const double log2h = (double)(31 - __clz(G / 2));
  const int bin = (int)floor((double)nbins * log2((double)n2) / (2.0 * log2h));
  return bin < nbins ? bin : -1;
}

template <typename R, int G>
__device__ __forceinline__ double mode_power(const PkArgs& a, size_t gi) {
  const size_t plane = (size_t)G * G * (G / 2);
  const cplx<R>* scr = (const cplx<R>*)a.scratch;
  const cplx<R> u = scr[a.bin_plane * plane + gi];
  const cplx<R> v = a.auto_mode ? u : scr[(a.bin_plane + 1) * plane + gi];
  const double norm = a.volume / ((double)G * G * G * (double)G * G * G);
  return norm * ((double)u.x * (double)v.x + (double)u.y * (double)v.y);
}

template <typename R, int G>
__global__ void __launch_bounds__(256) k_bin_max(PkArgs a) {
  const size_t plane = (size_t)G * G * (G / 2);
  float m = 0.0f;
  for (size_t gi = blockIdx.x * (size_t)blockDim.x + threadIdx.x; gi < plane;
       gi += (size_t)gridDim.x * blockDim.x) {
    long n2;
    int nz;
    if (mode_bin(gi, G, a.nbins, &n2, &nz) < 0) continue;
    m = fmaxf(m, __double2float_ru(fabs(mode_power<R, G>(a, gi))));
  }
  block_max_bits(m, a.max_bits);
}

// 128-bit add of a signed 64-bit value into (lo, hi) words.
__device__ __forceinline__ void add128(unsigned long long* lo, unsigned long long* hi, long long v) {
  const unsigned long long u = (unsigned long long)v;
  const unsigned long long old = atomicAdd(lo, u);
  const unsigned long long carry = (old + u < old) ? 1ull : 0ull;
  const unsigned long long h = (v < 0 ? ~0ull : 0ull) + carry;
  if (h) atomicAdd(hi, h);
}

constexpr double kNScale = 1125899906842624.0;   // 2^50: units of the |n| sums

template <typename R, int G>
__global__ void __launch_bounds__(256) k_bin_fixed(PkArgs a) {
  __shared__ unsigned long long acc[5 * 256];
  const int nb = a.nbins;
  const size_t plane = (size_t)G * G * (G / 2);
  for (int e = threadIdx.x; e < 5 * nb; e += blockDim.x) acc[e] = 0;
  __syncthreads();
  int e2;
  frexpf(__uint_as_float(*a.max_bits), &e2);       // every |P| < 2^e2
  const double inv_q = ldexp(1.0, 61 - e2);
  for (size_t gi = blockIdx.x * (size_t)blockDim.x + threadIdx.x; gi < plane;
       gi += (size_t)gridDim.x * blockDim.x) {
    long n2;
    int nz;
    const int bin = mode_bin(gi, G, nb, &n2, &nz);
    if (bin < 0) continue;
    const long long w = nz == 0 ? 1 : 2;
    const long long pq = __double2ll_rn(mode_power<R, G>(a, gi) * inv_q) * w;
    const long long nq = __double2ll_rn(sqrt((double)n2) * kNScale) * w;
    atomicAdd(&acc[bin], (unsigned long long)w);
    add128(&acc[nb + bin], &acc[2 * nb + bin], nq);
    add128(&acc[3 * nb + bin], &acc[4 * nb + bin], pq);
  }
  __syncthreads();
  for (int b = threadIdx.x; b < nb; b += blockDim.x) {
    if (!acc[b]) continue;
    atomicAdd(&a.acc[b], acc[b]);
    for (int k = 0; k < 2; ++k) {   // 128-bit block sums into the global ones
      const unsigned long long lo = acc[(1 + 2 * k) * nb + b], hi = acc[(2 + 2 * k) * nb + b];
      const unsigned long long old = atomicAdd(&a.acc[(1 + 2 * k) * nb + b], lo);
      const unsigned long long h = hi + ((old + lo < old) ? 1ull : 0ull);
      if (h) atomicAdd(&a.acc[(2 + 2 * k) * nb + b], h);
    }
  }
  // the block that adds last turns the exact sums into binary64: bins gets
  // [count][sum |k|][sum P], means [mean |k|][mean P][count] where it is asked
  // for (NaN for an empty bin).  The sums are only ever touched by agent-scope
  // atomics, which bypass the caches: they need no cache write-back (a release
  // fence) before the ticket, only to have been carried out.
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  __shared__ bool last;
  if (threadIdx.x == 0) last = atomicAdd(a.ticket, 1u) == gridDim.x - 1;
  __syncthreads();
  if (!last) return;
  const double q = ldexp(1.0, e2 - 61);
  auto sum = [&](int k) { return __hip_atomic_load(&a.acc[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
  for (int b = threadIdx.x; b < nb; b += blockDim.x) {
    const double nsum = ((double)sum(2 * nb + b) * 18446744073709551616.0 + (double)sum(nb + b)) / kNScale;
    const double psum = ((double)(long long)sum(4 * nb + b) * 18446744073709551616.0 +
                         (double)sum(3 * nb + b)) * q;
    const double cnt = (double)sum(b), ksum = a.kf * nsum;
    a.bins[b] = cnt;
    a.bins[nb + b] = ksum;
    a.bins[2 * nb + b] = psum;
    if (a.means) {
      const double nan = __longlong_as_double(0x7ff8000000000000LL);
      a.means[b] = cnt > 0 ? ksum / cnt : nan;
      a.means[nb + b] = cnt > 0 ? psum / cnt : nan;
      a.means[2 * nb + b] = cnt;
    }
  }
}

// bfloat16 meshes: one block = 2 x-values by 4 y-lines (8 z-lines), so that
// it writes whole halves of 4^3-cell bricks (32 cells of 2 NSLOT bytes: whole
// 128-byte lines, vector stores per cell) instead of fragments of lines
// shared with blocks on other XCDs.  M threads hold one field's 8 lines, 8
// elements each (8 threads, 4 elements for M = 4), and F fields are transformed
// at a time, so that every thread has a butterfly in the radix-8 stages; the
// next fields' lines are loaded meanwhile.  The results are staged as bfloat16
// pairs (the same rounding as the per-cell stores above) in per-slot rows
// padded to spread the 8 lines
// over the banks.  7 slots of 256^3 (0.74 GB): 298 us with a field at a time
// (half of the threads idle in the radix-8 stages, nine barriers per field, and
// reads of 8 lines per wave instead of 512 bytes of one), 165 us, the rate of a
// copy.  6 slots of 512^3: 1.94 -> 1.34 ms.
template <int NSLOT> struct CellWords;
template <> struct CellWords<8> { using T = uint4; };
template <> struct CellWords<6> { using T = uint3; };
template <> struct CellWords<4> { using T = uint2; };

template <int G> struct BfShape {
  static constexpr int M = G / 2, NL = 8;
  static constexpr int T = M < NL ? NL : M;                // threads per field
  static constexpr int F0 = 256 / T;
  static constexpr int F = F0 > 8 ? 8 : F0 < 2 ? 2 : F0;   // fields at a time
  static constexpr int NT = T * F;
};

template <int G, int NSLOT>
__global__ void __launch_bounds__(BfShape<G>::NT) k_zpass_c2r_bf16(GridBuildArgs a) {
  using R = float;
  using S = BfShape<G>;
  constexpr int M = S::M, NL = S::NL, NT = S::NT, T = S::T, F = S::F, H = M / 2;
  constexpr int PP = H * NL / T;                    // pairs (k, M - k) per thread
  using L = Lines<R, M, NL, T, true, 2, true, true>;
  constexpr int SW = (G + 16) / 2;                  // 32-bit words per staged row (line, slot)
  __shared__ cplx<R> lines[F * M * NL];
  __shared__ uint32_t stage[NSLOT * NL * SW];
  const int nyb = G / 4;
  const int ix0 = (blockIdx.x / nyb) * 2, iy0 = (blockIdx.x % nyb) * 4;
  const cplx<R>* __restrict__ twiddle = (const cplx<R>*)a.twiddle;
  const size_t plane = (size_t)G * G * M;
  const int tf = threadIdx.x % T, f0 = threadIdx.x / T;
  cplx<R>* const buf = lines + f0 * (M * NL);
  // a thread's pairs (k, m): the same k in every T/H-th line; line
  // l = 4 (x offset) + (y offset)
  const int k = tf % H, m = k ? M - k : H;
  const cplx<R> wk = twiddle[k], wm = twiddle[m];
  const typename L::Twiddles tw(twiddle, tf);
  const cplx<R>* const scr = (const cplx<R>*)a.scratch + ((size_t)ix0 * G + iy0) * M;
  cplx<R> xk[PP], xm[PP];
  auto load = [&](int f) {
    if (f >= a.nfft) return;
#pragma unroll
    for (int p = 0; p < PP; ++p) {
      const int line = tf / H + (T / H) * p;
      const cplx<R>* const src = scr + f * plane + ((size_t)(line >> 2) * G + (line & 3)) * M;
      xk[p] = src[k];
      xm[p] = src[m];
    }
  };
  load(f0);
  for (int e = threadIdx.x; e < NSLOT * NL * SW; e += NT) stage[e] = 0u;
  lds_barrier();
#pragma unroll 1
  for (int fb = 0; fb < a.nfft; fb += F) {
    const int f = fb + f0;
#pragma unroll
    for (int p = 0; p < PP; ++p) {
      const int line = tf / H + (T / H) * p;
      buf[L::at(k, line)] = c2r_element(xk[p], k ? xm[p] : cplx<R>{0.f, 0.f}, wk);
      buf[L::at(m, line)] = c2r_element(xm[p], k ? xk[p] : xm[p], wm);
    }
    load(f + F);
    lds_barrier();
    cplx<R> v[L::E];
    L::first(v, tf, buf);
    lds_barrier();
    const int slot = f < a.nfft ? a.slot[f] : -1;
    L::run(v, tf, buf, tw, [&](int dn, cplx<R> z) {
      if (slot >= 0) stage[(slot * NL + tf % NL) * SW + tf / NL + dn] = f32_to_bf16_bits(z.x) | (f32_to_bf16_bits(z.y) << 16);
    });
  }
  lds_barrier();
  // brick j along z: cells base(j) + c, c = 16 dx + 4 dy + dz in [0, 32), two at a time
  using W = typename CellWords<NSLOT>::T;
  W* out = (W*)a.out;
  const size_t base0 = (size_t)mesh_x(ix0, G) + mesh_y(iy0, G);
#pragma unroll 2
  for (int t = threadIdx.x; t < (G / 4) * 16; t += NT) {
    const int j = t >> 4, c = (t & 15) * 2;
    const int line = (c >> 4) * 4 + ((c >> 2) & 3);
    const uint32_t* const st = stage + line * SW + 2 * j + ((c & 3) >> 1);
    uint32_t lo[NSLOT / 2], hi[NSLOT / 2];
#pragma unroll
    for (int q = 0; q < NSLOT / 2; ++q) {
      const uint32_t w0 = st[(2 * q) * NL * SW], w1 = st[(2 * q + 1) * NL * SW];
      lo[q] = (w0 & 0xFFFFu) | (w1 << 16);
      hi[q] = (w0 >> 16) | (w1 & 0xFFFF0000u);
    }
    W* const o = out + base0 + mesh_z(4 * j) + c;
    if constexpr (NSLOT == 8) { o[0] = make_uint4(lo[0], lo[1], lo[2], lo[3]); o[1] = make_uint4(hi[0], hi[1], hi[2], hi[3]); }
    else if constexpr (NSLOT == 6) { o[0] = make_uint3(lo[0], lo[1], lo[2]); o[1] = make_uint3(hi[0], hi[1], hi[2]); }
    else { o[0] = make_uint2(lo[0], lo[1]); o[1] = make_uint2(hi[0], hi[1]); }
  }
}

// --------------------------------------------------------------- dispatch --
template <typename R, int G>
void build_grids_g(const GridBuildArgs& a, hipStream_t s) {
  using S = Shape<R, G>;
  const int nzb = S::M / S::NBC;
  hipLaunchKernelGGL((k_xpass_inverse<R, G>), dim3(G * nzb), dim3(S::NTX), 0, s, a);
  hipLaunchKernelGGL((k_ypass<R, G, true>), dim3(a.nfft * G * nzb), dim3(S::NTS), 0, s,
                     (cplx<R>*)a.scratch, (const cplx<R>*)a.twiddle);
  const int nyb = G / S::NL;
  const dim3 zg(G * nyb);
  if constexpr (std::is_same<R, float>::value) {
    if constexpr (G <= 512) {   // the staged outputs of 8 lines fit in LDS
      if (a.out_type == GT_BF16) {
        const dim3 zb((G / 2) * (G / 4));
        if (a.nslot == 8) hipLaunchKernelGGL((k_zpass_c2r_bf16<G, 8>), zb, dim3(BfShape<G>::NT), 0, s, a);
        else if (a.nslot == 6) hipLaunchKernelGGL((k_zpass_c2r_bf16<G, 6>), zb, dim3(BfShape<G>::NT), 0, s, a);
        else hipLaunchKernelGGL((k_zpass_c2r_bf16<G, 4>), zb, dim3(BfShape<G>::NT), 0, s, a);
        return;
      }
    }
    if (a.out_type == GT_BF16) {
      if (a.nslot == 8) hipLaunchKernelGGL((k_zpass_c2r<R, G, 8, GT_BF16>), zg, dim3(S::NT), 0, s, a);
      else if (a.nslot == 6) hipLaunchKernelGGL((k_zpass_c2r<R, G, 6, GT_BF16>), zg, dim3(S::NT), 0, s, a);
      else hipLaunchKernelGGL((k_zpass_c2r<R, G, 4, GT_BF16>), zg, dim3(S::NT), 0, s, a);
    } else {
      if (a.nslot == 8) hipLaunchKernelGGL((k_zpass_c2r<R, G, 8, GT_F32>), zg, dim3(S::NT), 0, s, a);
      else hipLaunchKernelGGL((k_zpass_c2r<R, G, 4, GT_F32>), zg, dim3(S::NT), 0, s, a);
    }
  } else {
    if (a.nslot == 8) hipLaunchKernelGGL((k_zpass_c2r<R, G, 8, GT_F64>), zg, dim3(S::NT), 0, s, a);
    else if (a.nslot == 6) hipLaunchKernelGGL((k_zpass_c2r<R, G, 6, GT_F64>), zg, dim3(S::NT), 0, s, a);
    else hipLaunchKernelGGL((k_zpass_c2r<R, G, 4, GT_F64>), zg, dim3(S::NT), 0, s, a);
  }
}

template <typename R, int G>
void power_spectrum_g(const PkArgs& a, hipStream_t s) {
  using S = Shape<R, G>;
  const int halves = a.auto_mode ? 1 : 2;
  const int nyb = G / S::NL;
  hipLaunchKernelGGL((k_zpass_r2c<R, G>), dim3(halves * G * nyb), dim3(S::NT), 0, s, a);
  const int nzb = S::M / S::NBC;
  hipLaunchKernelGGL((k_ypass<R, G, false>), dim3(halves * G * nzb), dim3(S::NTS), 0, s,
                     (cplx<R>*)a.scratch, (const cplx<R>*)a.twiddle);
  hipLaunchKernelGGL((k_xpass_accum<R, G>), dim3(halves * G * nzb), dim3(S::NTS), 0, s, a);
}

template <typename R, int G>
void bin_g(const PkArgs& a, hipStream_t s) {
  const size_t plane = (size_t)G * G * (G / 2);
  const size_t blocks = std::min<size_t>((plane + 255) / 256, 2048);
  hipLaunchKernelGGL((k_bin_max<R, G>), dim3((unsigned)blocks), dim3(256), 0, s, a);
  hipLaunchKernelGGL((k_bin_fixed<R, G>), dim3((unsigned)blocks), dim3(256), 0, s, a);
}

template <typename R>
void build_grids_r(const GridBuildArgs& a, hipStream_t s) {
  switch (a.G) {
    case 8: build_grids_g<R, 8>(a, s); break;
    case 16: build_grids_g<R, 16>(a, s); break;
    case 32: build_grids_g<R, 32>(a, s); break;
    case 64: build_grids_g<R, 64>(a, s); break;
    case 128: build_grids_g<R, 128>(a, s); break;
    case 256: build_grids_g<R, 256>(a, s); break;
    case 512: build_grids_g<R, 512>(a, s); break;
    case 1024: build_grids_g<R, 1024>(a, s); break;
    default: break;
  }
}

template <typename R>
void bin_r(const PkArgs& a, hipStream_t s) {
  switch (a.G) {
    case 8: bin_g<R, 8>(a, s); break;
    case 16: bin_g<R, 16>(a, s); break;
    case 32: bin_g<R, 32>(a, s); break;
    case 64: bin_g<R, 64>(a, s); break;
    case 128: bin_g<R, 128>(a, s); break;
    case 256: bin_g<R, 256>(a, s); break;
    case 512: bin_g<R, 512>(a, s); break;
    case 1024: bin_g<R, 1024>(a, s); break;
    default: break;
  }
}

template <typename R>
void power_spectrum_r(const PkArgs& a, hipStream_t s) {
  switch (a.G) {
    case 8: power_spectrum_g<R, 8>(a, s); break;
    case 16: power_spectrum_g<R, 16>(a, s); break;
    case 32: power_spectrum_g<R, 32>(a, s); break;
    case 64: power_spectrum_g<R, 64>(a, s); break;
    case 128: power_spectrum_g<R, 128>(a, s); break;
    case 256: power_spectrum_g<R, 256>(a, s); break;
    case 512: power_spectrum_g<R, 512>(a, s); break;
    case 1024: power_spectrum_g<R, 1024>(a, s); break;
    default: break;
  }
}

}  // namespace

void launch_build_grids(const GridBuildArgs& a, hipStream_t s) {
  if (a.fp64) build_grids_r<double>(a, s);
  else build_grids_r<float>(a, s);
}

void launch_power_spectrum(const PkArgs& a, hipStream_t s) {
  if (a.fp64) power_spectrum_r<double>(a, s);
  else power_spectrum_r<float>(a, s);
}

void launch_bin(const PkArgs& a, hipStream_t s) {
  if (a.fp64) bin_r<double>(a, s);
  else bin_r<float>(a, s);
}

}  // namespace fdf
