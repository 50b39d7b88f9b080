// Host runtime and C ABI of the FastDF push (see include/fastdf.h).
//
// Host work is FP64 bookkeeping: configuration checks, the constant-Delta-log-a
// schedule with its conformal-time integrals (sec. 3.3), the sigma_8
// normalisation of the seeded field, <eps>(a) for the density estimator
// (sec. 2.2), carving the caller's workspace, and enqueuing kernels.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "../../include/fastdf.h"
#include "fdf_internal.h"

using namespace fdf;

namespace {

constexpr double kCkms = 299792.458;          // speed of light [km/s]
constexpr double kBoltzmannEvK = 8.617333262e-5;
constexpr double kTnuKelvin = 1.95;           // present neutrino temperature (sec. 2)
constexpr double kPi = 3.14159265358979323846;
constexpr int kMaxBins = 256;
// Spectrum bins region: [3][kMaxBins] binary64 results, then the exact sums
// [5][kMaxBins] (64-bit words), then the largest |P| word and the ticket.
constexpr size_t kBinsBytes = (8 * kMaxBins + 2) * 8;
constexpr size_t kAlign = 256;

double t_nu_ev() { return kTnuKelvin * kBoltzmannEvK; }
size_t align_up(size_t v) { return (v + kAlign - 1) / kAlign * kAlign; }

// ---------------------------------------------------------------- quadrature --
struct GaussLegendre {
  double x[16], w[16];
  GaussLegendre() {
    // nodes of P_16 by Newton's method on the Legendre recurrence
    const int n = 16;
    for (int i = 0; i < n; ++i) {
      long double z = cosl(kPi * (i + 0.75L) / (n + 0.5L)), pp = 0;
      for (int it = 0; it < 100; ++it) {
        long double p1 = 1, p2 = 0;
        for (int j = 1; j <= n; ++j) {
          long double p3 = p2;
          p2 = p1;
          p1 = ((2 * j - 1) * z * p2 - (j - 1) * p3) / j;
        }
        pp = n * (z * p1 - p2) / (z * z - 1);
        long double dz = p1 / pp;
        z -= dz;
        if (fabsl(dz) < 1e-19L) break;
      }
      x[i] = (double)z;
      w[i] = (double)(2 / ((1 - z * z) * pp * pp));
    }
  }
  template <class F> double integrate(F f, double lo, double hi, int panels) const {
    long double sum = 0;
    const double h = (hi - lo) / panels;
    for (int p = 0; p < panels; ++p) {
      const double c = lo + (p + 0.5) * h, r = 0.5 * h;
      for (int i = 0; i < 16; ++i) sum += (long double)w[i] * r * f(c + r * x[i]);
    }
    return (double)sum;
  }
};
const GaussLegendre& gl16() { static GaussLegendre g; return g; }

struct Cosmo {
  double h, om, orad, ol;
  double H0() const { return 100.0 * h / kCkms; }
  double H(double a) const { return H0() * std::sqrt(orad / (a * a * a * a) + om / (a * a * a) + ol); }
};

// Delta tau = int_{ln a0}^{ln a1} dln a / (a H)  (sec. 3.3, step sizes)
double dtau(const Cosmo& c, double lna0, double lna1) {
  const int panels = std::max(1, (int)std::ceil(std::fabs(lna1 - lna0) / 0.02));
  return gl16().integrate([&](double l) { const double a = std::exp(l); return 1.0 / (a * c.H(a)); },
                          lna0, lna1, panels);
}

// tau(a) from a = 0 (the integrand vanishes like a^(1/2) or a as a -> 0)
double conformal_time(const Cosmo& c, double a) {
  const double l1 = std::log(a), l0 = l1 - 80.0;
  return dtau(c, l0, l1);
}

double bbks(double k, double gamma, double h) {
  const double q = k / (gamma * h);
  if (q <= 0) return 1.0;
  const double b = 16.1 * q, cc = 5.46 * q, d = 6.71 * q;
  const double poly = 1.0 + 3.89 * q + b * b + cc * cc * cc + (d * d) * (d * d);
  return std::log1p(2.34 * q) / (2.34 * q) * std::pow(poly, -0.25);
}

double tophat(double x) {
  if (std::fabs(x) < 0.1) {
    const double x2 = x * x;
    return 1.0 - x2 / 10.0 + x2 * x2 / 280.0 - x2 * x2 * x2 / 15120.0 + x2 * x2 * x2 * x2 / 1330560.0;
  }
  return 3.0 * (std::sin(x) - x * std::cos(x)) / (x * x * x);
}

// A with sigma(8 Mpc/h) = sigma8 for P = A k^ns T_BBKS^2
double power_amplitude(double sigma8, double ns, double gamma, double h) {
  const double R = 8.0 / h;
  auto f_lnk = [&](double l) {
    const double k = std::exp(l), t = bbks(k, gamma, h), w = tophat(k * R);
    return k * k * k * std::pow(k, ns) * t * t * w * w;
  };
  auto f_k = [&](double k) {
    const double t = bbks(k, gamma, h), w = tophat(k * R);
    return k * k * std::pow(k, ns) * t * t * w * w;
  };
  double s2 = gl16().integrate(f_lnk, std::log(1e-7), 0.0, 400);
  s2 += gl16().integrate(f_k, 1.0, 1000.0, 20000);
  s2 /= 2.0 * kPi * kPi;
  return sigma8 * sigma8 / s2;
}

// int_0^64 f(x) dx over panels that double in width from 2^-12: an integrand
// like x^2 sqrt(x^2 + s^2) / (1 + e^x) varies on the scale of x (or of 1) for
// every s, so 16 points on each of the 19 panels leave binary64 rounding alone.
template <class F> double integrate_doubling(F f) {
  double sum = gl16().integrate(f, 0.0, 0x1p-12, 1);
  for (double lo = 0x1p-12; lo < 64.0; lo *= 2.0) sum += gl16().integrate(f, lo, 2.0 * lo, 1);
  return sum;
}

// <eps>(a) = int q^2 sqrt(q^2 + m^2 a^2) fbar / int q^2 fbar  (eq. rho_def normalisation)
double mean_energy(double m, double a) {
  const double T = t_nu_ev(), ma = m * a;
  static const double den = integrate_doubling([](double x) { return x * x / (1.0 + std::exp(x)); });
  return integrate_doubling([&](double x) { return x * x * std::sqrt(x * x * T * T + ma * ma) / (1.0 + std::exp(x)); }) /
         den;
}

// Radiation-to-matter potential factor g(a) = (10/9) Phi(y)/Phi(0), y = a/a_eq,
// Phi(y)/Phi(0) = 1 - y (s^2 + 4 s + 5) / (10 (s+1)^4), s = sqrt(1+y)
// (Kodama-Sasaki super-horizon solution without cancellation), and dg/da.
void radmat_factor(double a, double om, double orad, double* g, double* dg) {
  const double aeq = orad / om, y = a / aeq, s = std::sqrt(1.0 + y);
  const double num = y + 6.0 + 4.0 * s, den = std::pow(s + 1.0, 4);
  const double hfun = y * num / den;
  const double dnum = 1.0 + 2.0 / s, dden = 4.0 * std::pow(s + 1.0, 3) / (2.0 * s);
  const double dh = (num + y * dnum) / den - y * num * dden / (den * den);
  *g = (10.0 / 9.0) * (1.0 - hfun / 10.0);
  *dg = -(1.0 / 9.0) * dh / aeq;
}

bool is_pow2(int v) { return v > 0 && (v & (v - 1)) == 0; }
int ilog2(int v) { int r = 0; while ((1 << r) < v) ++r; return r; }

// ----------------------------------------------------------------- layout --
struct Layout {
  size_t twiddle_d, twiddle_f, seg, bins, dep, scratch, dens, fields, parts, sort_count, sort_scan, sort_rank,
      sort_bucket, sort_src, sort_key, total;
  int64_t sort_keys_max;
  int grid_sets;
  size_t field_dk_bytes, field_grid_bytes, scratch_bytes, dens_bytes, parts_bytes;
  int nslot;
};

bool eom_potentials(const fdf_config& c) { return c.eom == FDF_EOM_EXACT || c.eom == FDF_EOM_CANONICAL; }
// Slots per mesh cell.  Separable form: grad psi and phi-dot (4) when
// psi = phi; else grad psi, grad phi and phi-dot (8).  When phi-dot is zero
// the cell drops it and the pad: 6 slots (binary64: three 16-byte loads per
// corner; bfloat16: one 12-byte load), unless pad_mesh asks for the aligned
// 16-byte bfloat16 cell.
int slots_for(const fdf_config& c) {
  if (c.eom == FDF_EOM_SEPARABLE) {
    if (c.slip_amp == 0.0) return 4;
    const bool f64 = c.precision == FDF_PREC_FP64;
    if (c.potential_model == FDF_MODEL_RADMAT) return 8;
    return (f64 || !c.pad_mesh) ? 6 : 8;
  }
  return eom_potentials(c) ? 8 : 4;
}
int fft_planes(const fdf_config& c) { return eom_potentials(c) ? 8 : 7; }

// Stored slot of a grid quantity (0-2 grad psi, 3-5 grad phi, 6 phi-dot,
// 7 psi, 8 phi, 9 phi + psi): >= 0 the slot, -1 identically zero in this
// configuration, -2 not stored for this equation of motion.
int grid_slot(const fdf_config& c, int quantity) {
  const bool tdep = c.potential_model == FDF_MODEL_RADMAT;
  const bool same = c.slip_amp == 0.0;   // phi = psi
  switch (c.eom) {
    case FDF_EOM_SEPARABLE:
      if (slots_for(c) == 8) return quantity <= 5 ? quantity : quantity == 6 ? (tdep ? 6 : -1) : -2;
      if (slots_for(c) == 6) return quantity <= 5 ? quantity : quantity == 6 ? -1 : -2;
      if (quantity <= 5) return quantity % 3;
      return quantity == 6 ? (tdep ? 3 : -1) : -2;
    case FDF_EOM_EXACT:
      if (quantity <= 5) return quantity;
      return quantity == 6 ? (tdep ? 6 : -1) : quantity == 9 ? 7 : -2;
    case FDF_EOM_CANONICAL:
      if (quantity <= 5) return quantity;
      return quantity == 7 ? 6 : quantity == 8 ? 7 : -2;
    default:
      if (quantity <= 2) return quantity;
      return (quantity <= 5 && same) ? quantity - 3 : -2;
  }
}
size_t real_bytes(const fdf_config& c) { return c.precision == FDF_PREC_FP64 ? 8 : 4; }
size_t slot_bytes(const fdf_config& c) { return c.precision == FDF_PREC_FP64 ? 8 : 2; }
size_t particle_bytes(const fdf_config& c) { return c.precision == FDF_PREC_FP64 ? 76 : 40; }
int arrays_per_species(const fdf_config& c) { return c.precision == FDF_PREC_FP64 ? 10 : 10; }

Layout plan(const fdf_config& c) {
  Layout L{};
  const size_t G = (size_t)c.grid_n, rb = real_bytes(c), cb = 2 * rb;
  L.nslot = slots_for(c);
  L.field_dk_bytes = align_up(G * G * (G / 2) * cb);
  L.field_grid_bytes = align_up(G * G * G * (size_t)L.nslot * slot_bytes(c));
  L.scratch_bytes = align_up((size_t)fft_planes(c) * G * G * (G / 2) * cb);
  L.dens_bytes = align_up(4 * G * G * G * rb);   // two halves, or a 4-slot pre-IC grid
  const int copies = c.sort_every > 0 ? 2 : 1;
  L.parts_bytes = align_up((size_t)c.max_particles * particle_bytes(c) * copies +
                           (size_t)c.max_species * arrays_per_species(c) * copies * kAlign);
  size_t off = 0;
  // twiddles of the G-point transform, then those of G/2, G/4, ... 8 (the
  // analysis meshes of the spectra): the table of n points starts at entry 2 (G - n)
  L.twiddle_d = off; off += align_up(2 * G * 16);
  L.twiddle_f = off; off += align_up(2 * G * 8);
  L.seg = off; off += 2 * align_up((size_t)c.max_species * sizeof(Segment));
  L.bins = off; off += align_up(kBinsBytes);
  L.dep = off; off += kAlign;   // the fixed-point deposit's largest |value|
  L.scratch = off; off += L.scratch_bytes;
  L.dens = off; off += L.dens_bytes;
  L.grid_sets = (c.potential_model == FDF_MODEL_RADMAT && c.superstep_tol > 0) ? 2 : 1;
  L.fields = off; off += (size_t)c.max_fields * (L.field_dk_bytes + L.grid_sets * L.field_grid_bytes);
  L.parts = off; off += L.parts_bytes;
  const int64_t tmax = std::min<int64_t>(c.grid_n, 256);
  const bool sorting = c.sort_every > 0;
  L.sort_keys_max = sorting ? tmax * tmax * tmax : 0;
  L.sort_count = off; off += align_up((size_t)L.sort_keys_max * 4);
  L.sort_scan = off; off += sorting ? align_up(sort_scan_scratch_words(L.sort_keys_max) * 4) : 0;
  L.sort_rank = off; off += sorting ? align_up((size_t)c.max_particles * 4) : 0;
  L.sort_bucket = off; off += sorting ? align_up((size_t)c.max_particles * 4) : 0;
  L.sort_src = off; off += sorting ? align_up((size_t)c.max_particles * 4) : 0;
  L.sort_key = off; off += sorting ? align_up((size_t)c.max_particles * 4) : 0;
  L.total = off;
  return L;
}

const char* validate(const fdf_config* c) {
  if (!c) return "config is NULL";
  if (c->abi_version != FDF_ABI_VERSION) return "abi_version mismatch";
  if (!is_pow2(c->grid_n) || c->grid_n < 8 || c->grid_n > 1024) return "grid_n must be a power of two in [8, 1024]";
  if (!(c->box_mpc > 0) || !std::isfinite(c->box_mpc)) return "box_mpc must be positive";
  if (!(c->h > 0)) return "h must be positive";
  if (c->omega_m < 0 || c->omega_r < 0 || c->omega_l < 0 || c->omega_m + c->omega_r <= 0)
    return "need omega_m + omega_r > 0 and non-negative densities";
  if (!(c->z_begin > -1) || !(c->z_end > -1)) return "redshifts must exceed -1";
  if (c->z_begin == c->z_end) return "z_begin must differ from z_end";
  if (c->n_steps < 1) return "n_steps must be >= 1";
  if (c->precision != FDF_PREC_FP64 && c->precision != FDF_PREC_FP32) return "unknown precision";
  if (c->potential_model != FDF_MODEL_POISSON && c->potential_model != FDF_MODEL_RADMAT) return "unknown potential model";
  if (c->potential_model == FDF_MODEL_RADMAT && !(c->omega_r > 0)) return "RADMAT needs omega_r > 0";
  if (c->slip_amp < 0 || c->slip_amp >= 1 || !(c->slip_k > 0)) return "slip_amp in [0,1) and slip_k > 0 required";
  if (!(c->sigma8 > 0) || !(c->gamma > 0)) return "sigma8 and gamma must be positive";
  if (c->sort_every < 0) return "sort_every must be >= 0";
  if (c->max_fields < 1 || c->max_species < 1 || c->max_particles < 1) return "capacities must be >= 1";
  if (c->max_particles > ((int64_t)1 << 32)) return "at most 2^32 particles";
  if (!(c->superstep_tol >= 0) || !std::isfinite(c->superstep_tol)) return "superstep_tol must be >= 0";
  if (c->eom < FDF_EOM_SEPARABLE || c->eom > FDF_EOM_NEWTONIAN) return "unknown equation of motion";
  if (c->interp_order < 0 || c->interp_order > 2) return "interp_order must be 0, 1 (CIC) or 2 (TSC)";
  if (c->pad_mesh != 0 && c->pad_mesh != 1) return "pad_mesh must be 0 or 1";
  return nullptr;
}

struct FieldRec {
  uint64_t seed = 0;
  void* dk = nullptr;
  void* grid = nullptr;
  void* grid2 = nullptr;      // second grid set (super-steps)
  bool has_grid = false;
  double grid_a = 0;
  int tag[2] = {-1, -1};      // super-steps: anchor (schedule index) held by each set
};

enum { kThisCall = 1, kEarlierCall = 2 };

struct SpeciesRec {
  int field = 0;
  double m = 0;
  int64_t n = 0;
  uint64_t seed = 0;
  int flags = 0;
  Segment seg[2];   // state buffers (second copy only with sorting)
  int cur = 0;
  bool pristine = false;   // state is exactly the sampled one (no pre-IC, not stepped)
  bool sorted = false;     // in spatial order
  bool placed = false;     // that order is the one of its creation, without a prediction
  int order_time = -1;     // integer time from which its current order is meant to be used (-1: none)
  double drift_cells = 0;  // typical drift since that time, in mesh cells
  int waited = 0;          // its first order in place was left to a later call: kThisCall, kEarlierCall
};

// A captured step sequence: the host state it was captured from and the host
// state it leaves behind, so a replay can stand in for the enqueue.
struct HostStepState {
  int step_index = 0;
  std::vector<int> ints;           // per species: copy of its state, sorted, placed, order time,
                                   // pristine, waited; per field: two super-step set tags
  std::vector<double> drift_cells; // per species
  std::vector<double> grid_a;      // per field; NaN = no grid
  bool operator==(const HostStepState& o) const {
    auto same = [](const std::vector<double>& x, const std::vector<double>& y) {   // bitwise: NaN equals itself
      return x.size() == y.size() && (x.empty() || std::memcmp(x.data(), y.data(), x.size() * sizeof(double)) == 0);
    };
    return step_index == o.step_index && ints == o.ints && same(drift_cells, o.drift_cells) &&
           same(grid_a, o.grid_a);
  }
};

struct GraphRec {
  int n = 0;
  std::vector<double> layout;      // fields and species that fix every device pointer
  HostStepState before, after;
  bool builds_grids = false;       // overwrites the FFT scratch and with it the last density
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
};

struct TimingRec {
  std::vector<std::pair<hipEvent_t, hipEvent_t>> pending;
  std::vector<std::pair<hipEvent_t, hipEvent_t>> pool;
  double total_ms = 0;
  int64_t launches = 0;
  int64_t work[3] = {0, 0, 0};   // particle-updates with a drift, kick-only updates, mesh cells read
  int64_t passes[2] = {0, 0};    // particles whose state launches read and wrote, with a drift and kick-only
};

}  // namespace

struct fdf_ctx {
  fdf_config cfg{};
  Cosmo cos{};
  hipStream_t stream = nullptr;
  std::vector<double> a, a_half, kick1, kick2, drift;
  std::vector<int> anchors;   // super-step anchors (schedule indices), empty when unused
  double amp = 0, tau_begin = 0;
  char* ws = nullptr;
  size_t ws_bytes = 0;
  Layout lay{};
  size_t field_next = 0, part_next = 0;
  std::vector<FieldRec> fields;
  std::vector<SpeciesRec> species;
  int step_index = 0;
  bool stepped = false;
  bool seg_dirty = true;
  int ppt = 4;
  int sort_tiles = 0;       // tiles per axis of the sort key (0: default)
  int sort_every = 0;       // current re-sort cadence
  float sort_cells = 0;     // adaptive cadence threshold in cells (0: fixed cadence)
  int persistent = 0;       // push grid size when > 0 (a multiple of 8)
  bool use_graph = false;   // capture step sequences into hipGraphs
  bool sort_predict = true; // sort keys from positions extrapolated to mid-interval
  bool sort_fused = true;   // FP32 separable: re-sorts after the first ride on the push
  int push_waves = 0;       // cap on resident push waves per SIMD (0: none)
  int sort_push_ppt = 4;    // particles per thread of the fused re-sort push
  bool sort_keys_push = true;   // the push before a re-sort writes the sort keys
  hipStream_t cap_stream = nullptr;   // private stream used only for graph capture
  hipStream_t launch_stream = nullptr;  // stream kernels are enqueued on right now
  std::vector<GraphRec> graphs;       // captured step sequences
  std::string err;
  bool timing = false;
  TimingRec tim[FDF_KERNEL_COUNT];
  bool have_density = false;
  int density_auto = 0;
  double* pinned = nullptr;   // 3 kMaxBins doubles of page-locked host memory for the spectra's bins
};

namespace {

int fail(fdf_ctx* c, int code, const std::string& msg) {
  if (c) c->err = msg;
  return code;
}

int hip_check(fdf_ctx* c, hipError_t e, const char* what) {
  if (e == hipSuccess) return FDF_OK;
  return fail(c, FDF_ERR_HIP, std::string(what) + ": " + hipGetErrorString(e));
}

int launched(fdf_ctx* c, const char* what) { return hip_check(c, hipGetLastError(), what); }

hipStream_t stream_of(fdf_ctx* c) { return c->launch_stream ? c->launch_stream : c->stream; }

void clear_graphs(fdf_ctx* c) {
  for (auto& g : c->graphs) {
    if (g.exec) (void)hipGraphExecDestroy(g.exec);
    if (g.graph) (void)hipGraphDestroy(g.graph);
  }
  c->graphs.clear();
}

void timing_begin(fdf_ctx* c, int cls, std::pair<hipEvent_t, hipEvent_t>* ev) {
  if (!c->timing || c->launch_stream) return;
  TimingRec& t = c->tim[cls];
  if (t.pool.empty()) {
    hipEvent_t e0, e1;
    (void)hipEventCreate(&e0);
    (void)hipEventCreate(&e1);
    t.pool.push_back({e0, e1});
  }
  *ev = t.pool.back();
  t.pool.pop_back();
  (void)hipEventRecord(ev->first, c->stream);
}

void timing_end(fdf_ctx* c, int cls, std::pair<hipEvent_t, hipEvent_t>& ev) {
  if (!c->timing || c->launch_stream) return;
  (void)hipEventRecord(ev.second, c->stream);
  c->tim[cls].pending.push_back(ev);
  c->tim[cls].launches++;
}

// Work done by the launches of a timed class (counted while timing is on).
void timing_work(fdf_ctx* c, int cls, int64_t particles, const PushStep* step, int nsteps, int64_t mesh_cells) {
  if (!c->timing || c->launch_stream) return;
  TimingRec& t = c->tim[cls];
  for (int s = 0; s < nsteps; ++s) t.work[step[s].do_drift ? 0 : 1] += particles;
  t.work[2] += mesh_cells;
  if (nsteps > 0) t.passes[step[0].do_drift ? 0 : 1] += particles;
}

void timing_collect(fdf_ctx* c) {
  for (auto& t : c->tim) {
    for (auto& ev : t.pending) {
      float ms = 0;
      (void)hipEventSynchronize(ev.second);
      (void)hipEventElapsedTime(&ms, ev.first, ev.second);
      t.total_ms += ms;
      t.pool.push_back(ev);
    }
    t.pending.clear();
  }
}

bool needs_ws(fdf_ctx* c) { return c->ws != nullptr; }

// Carve the state arrays of one copy of a species.
bool carve_species(fdf_ctx* c, Segment& s, int64_t n) {
  const bool f64 = c->cfg.precision == FDF_PREC_FP64;
  auto take = [&](size_t bytes) -> void* {
    const size_t sz = align_up(bytes);
    if (c->part_next + sz > c->lay.parts_bytes) return nullptr;
    void* p = c->ws + c->lay.parts + c->part_next;
    c->part_next += sz;
    return p;
  };
  std::memset(&s, 0, sizeof(s));
  for (int d = 0; d < 3; ++d) {
    if (f64) {
      s.xd[d] = (double*)take(n * 8);
      s.qd[d] = (double*)take(n * 8);
      s.q0d[d] = (double*)take(n * 8);
      if (!s.xd[d] || !s.qd[d] || !s.q0d[d]) return false;
    } else {
      s.xu[d] = (uint32_t*)take(n * 4);
      s.q0f[d] = (float*)take(n * 4);
      s.dqf[d] = (float*)take(n * 4);
      if (!s.xu[d] || !s.q0f[d] || !s.dqf[d]) return false;
    }
  }
  s.id = (uint32_t*)take(n * 4);
  s.n = n;
  return s.id != nullptr;
}

GridBuildArgs grid_recipe(fdf_ctx* c, const FieldRec& f, double a, bool pre_ic_grid) {
  GridBuildArgs g{};
  const fdf_config& cf = c->cfg;
  g.G = cf.grid_n;
  g.fp64 = cf.precision == FDF_PREC_FP64;
  g.kf = 2.0 * kPi / cf.box_mpc;
  const double base = -1.5 * c->cos.H0() * c->cos.H0() * cf.omega_m;   // Poisson: D(a)/a = 1
  double gf = 1.0, dgf = 0.0;
  if (cf.potential_model == FDF_MODEL_RADMAT) radmat_factor(a, cf.omega_m, cf.omega_r, &gf, &dgf);
  g.tr.c_phi = base * gf;
  g.tr.c_phidot = base * (a * a * c->cos.H(a) * dgf);
  g.tr.slip_amp = cf.slip_amp;
  g.tr.slip_k = cf.slip_k;
  g.delta_k = f.dk;
  g.scratch = c->ws + c->lay.scratch;
  g.twiddle = c->ws + (g.fp64 ? c->lay.twiddle_d : c->lay.twiddle_f);
  const bool phidot = cf.potential_model == FDF_MODEL_RADMAT;
  int n = 0;
  if (pre_ic_grid) {
    g.nslot = 4;
    g.out_type = g.fp64 ? GT_F64 : GT_F32;
    const int kinds[4] = {SK_DX_PSI, SK_DY_PSI, SK_DZ_PSI, SK_PSI};
    for (int i = 0; i < 4; ++i) { g.kind[n] = kinds[i]; g.slot[n] = i; ++n; }
    g.out = c->ws + c->lay.dens;
  } else {
    g.nslot = c->lay.nslot;
    g.out_type = g.fp64 ? GT_F64 : GT_BF16;
    g.out = f.grid;
    g.kind[n] = SK_DX_PSI; g.slot[n++] = 0;
    g.kind[n] = SK_DY_PSI; g.slot[n++] = 1;
    g.kind[n] = SK_DZ_PSI; g.slot[n++] = 2;
    if (cf.eom != FDF_EOM_SEPARABLE) {
      if (eom_potentials(cf)) {
        g.kind[n] = SK_DX_PHI; g.slot[n++] = 3;
        g.kind[n] = SK_DY_PHI; g.slot[n++] = 4;
        g.kind[n] = SK_DZ_PHI; g.slot[n++] = 5;
      }
      if (cf.eom == FDF_EOM_EXACT) {
        if (phidot) { g.kind[n] = SK_PHIDOT; g.slot[n++] = 6; }
        g.kind[n] = SK_PHI_PSI; g.slot[n++] = 7;
      } else if (cf.eom == FDF_EOM_CANONICAL) {
        g.kind[n] = SK_PSI; g.slot[n++] = 6;
        g.kind[n] = SK_PHI; g.slot[n++] = 7;
      }
    } else if (g.nslot >= 6) {
      g.kind[n] = SK_DX_PHI; g.slot[n++] = 3;
      g.kind[n] = SK_DY_PHI; g.slot[n++] = 4;
      g.kind[n] = SK_DZ_PHI; g.slot[n++] = 5;
      if (phidot) { g.kind[n] = SK_PHIDOT; g.slot[n++] = 6; }
    } else if (phidot) {
      g.kind[n] = SK_PHIDOT; g.slot[n++] = 3;
    }
  }
  g.nfft = n;
  return g;
}

int build_grid(fdf_ctx* c, int field, double a, int buf = 0) {
  FieldRec& f = c->fields[field];
  c->have_density = false;   // the FFT scratch holds the FP32 form's density copy
  GridBuildArgs g = grid_recipe(c, f, a, false);
  if (buf == 1) g.out = f.grid2;
  std::pair<hipEvent_t, hipEvent_t> ev;
  timing_begin(c, FDF_KERNEL_GRID, &ev);
  launch_build_grids(g, stream_of(c));
  timing_end(c, FDF_KERNEL_GRID, ev);
  if (buf == 0) {
    f.has_grid = true;
    f.grid_a = a;
  }
  return launched(c, "grid build");
}

// Two device tables of segments, one per buffer copy, stored by kernels from
// their arguments: nothing waits for the stream.
int upload_segments(fdf_ctx* c) {
  if (!c->seg_dirty) return FDF_OK;
  static_assert(sizeof(Segment) % 8 == 0, "whole words");
  const size_t table = align_up((size_t)c->cfg.max_species * sizeof(Segment));
  constexpr size_t per = kStoreWords * 8 / sizeof(Segment);
  StoreArgs st;
  for (int copy = 0; copy < 2; ++copy)
    for (size_t i = 0; i < c->species.size(); i += per) {
      const size_t n = std::min(per, c->species.size() - i);
      for (size_t k = 0; k < n; ++k) {
        const SpeciesRec& s = c->species[i + k];
        Segment g = s.seg[copy];
        g.grid = c->fields[s.field].grid;
        g.grid2 = c->fields[s.field].grid2;
        g.m = s.m;
        g.seed = s.seed;
        std::memcpy((char*)st.w + k * sizeof(Segment), &g, sizeof(g));
      }
      st.dst = (uint64_t*)(c->ws + c->lay.seg + copy * table + i * sizeof(Segment));
      st.n = (int32_t)(n * sizeof(Segment) / 8);
      launch_store(st, c->stream);
    }
  c->seg_dirty = false;
  return launched(c, "segment upload");
}

// LDS bytes per 4-wave push block that leave room for exactly `waves` blocks
// (one wave per SIMD each) in the 160 KB of a CU; 0 for no cap.
int push_lds_reserve(int waves) {
  if (waves <= 0) return 0;
  const int lds_per_cu = 160 * 1024;
  return (lds_per_cu / (waves + 1) + 256 + 255) / 256 * 256;
}

// Buckets per axis of the sort: default one per 4^3 cells, at most 256.
int sort_tiles_of(fdf_ctx* c) {
  const int tmax = std::min(c->cfg.grid_n, 256);
  int t = c->sort_tiles > 0 ? c->sort_tiles : std::max(1, c->cfg.grid_n / 4);
  return std::min(t, tmax);
}

// Drift of a mean-momentum particle (|q| = 3.151 T) of mass m over one drift
// of length dt at a, in mesh cells: the adaptive sort cadence of a species.
double typical_drift_cells(fdf_ctx* c, double dt, double a, double m) {
  const double q = 3.151374 * t_nu_ev();
  const double v = q / std::sqrt(q * q + m * m * a * a);
  return std::fabs(dt) * v * c->cfg.grid_n / c->cfg.box_mpc;
}

// Prediction of a re-sort: order by x + v tau at scale factor a_mid.
struct SortPrediction { double tau = 0, a_mid = 0; };

// Spatial re-sort of every species into its other buffer copy, ordered by
// the positions extrapolated by predict_tau at scale factor a_pred.
SortArgs sort_args(fdf_ctx* c, const SpeciesRec& s, double predict_tau, double a_pred) {
  const int tiles = sort_tiles_of(c);
  SortArgs a{};
  a.seg = s.seg[s.cur];
  a.dst = s.seg[s.cur ^ 1];
  a.predict_tau = predict_tau;
  a.ma = s.m * a_pred;
  a.fp64 = c->cfg.precision == FDF_PREC_FP64;
  a.grid_n = c->cfg.grid_n;
  a.cell_shift = 32 - ilog2(c->cfg.grid_n);
  a.fine_bits = ilog2(c->cfg.grid_n / tiles);
  a.box = c->cfg.box_mpc;
  a.nkeys = (int64_t)tiles * tiles * tiles;
  a.count = (uint32_t*)(c->ws + c->lay.sort_count);
  a.scan_scratch = (uint32_t*)(c->ws + c->lay.sort_scan);
  a.rank = (uint32_t*)(c->ws + c->lay.sort_rank);
  a.bucket = (uint32_t*)(c->ws + c->lay.sort_bucket);
  a.src = (uint32_t*)(c->ws + c->lay.sort_src);
  return a;
}

// Byte offset in the FFT scratch of the FP32 form's binary32 density halves:
// behind the four transform planes of the largest mesh (two halves and the
// momentum spectrum's two accumulators), 8 G^3 bytes, inside the scratch's
// 28 G^3 bytes.
size_t density_copy_offset(const fdf_ctx* c) {
  const size_t G = (size_t)c->cfg.grid_n;
  return 4 * (G * G * (G / 2)) * 8;
}

// Sampling of a species by the ids its segment g holds, within a step: the seed
// comes from the segment table, which is stored before every step.
SampleArgs resample_args(fdf_ctx* c, const SpeciesRec& s, const Segment& g) {
  SampleArgs sa{};
  sa.seg = g;
  sa.fp64 = c->cfg.precision == FDF_PREC_FP64;
  sa.by_id = 1;
  sa.seed_at = &((const Segment*)(c->ws + c->lay.seg))[&s - c->species.data()].seed;
  sa.box = c->cfg.box_mpc;
  sa.t_nu = t_nu_ev();
  return sa;
}

// A context without a second copy of the state re-orders it in place, through
// the FFT scratch, which is free between grid builds and spectra: the sort's
// lists and as many state arrays at a time as fit.  FP32: the lists lie in the
// fixed-point density halves and the arrays below the binary32 density copy, so
// that a density stays readable.
struct InPlaceRoom {
  char* lists = nullptr;
  size_t list_bytes = 0;
  char* arrays = nullptr;
  size_t array_bytes = 0;    // for state arrays at a time
};

// L2 of one XCD: a mesh it holds is gathered from at the same rate in any order.
constexpr size_t kL2Bytes = (size_t)4 << 20;

bool in_place_room(fdf_ctx* c, int64_t n, InPlaceRoom* r) {
  if (c->cfg.sort_every > 0 || c->lay.field_grid_bytes <= kL2Bytes) return false;
  const int64_t tiles = sort_tiles_of(c), nkeys = tiles * tiles * tiles;
  r->list_bytes = align_up(nkeys * 4) + align_up(sort_scan_scratch_words(nkeys) * 4) + 3 * align_up(n * 4);
  if (c->cfg.precision == FDF_PREC_FP64) {
    if (r->list_bytes > c->lay.scratch_bytes) return false;
    r->lists = c->ws + c->lay.scratch;
    r->arrays = r->lists + r->list_bytes;
    r->array_bytes = c->lay.scratch_bytes - r->list_bytes;
    return r->array_bytes >= align_up(n * 8);
  }
  if (r->list_bytes > c->lay.dens_bytes) return false;
  r->lists = c->ws + c->lay.dens;
  r->arrays = c->ws + c->lay.scratch;
  r->array_bytes = density_copy_offset(c);
  return r->array_bytes >= align_up(n * 4);
}

int sort_in_place(fdf_ctx* c, SpeciesRec& s, const SortPrediction& pred, const InPlaceRoom& room) {
  const bool f64 = c->cfg.precision == FDF_PREC_FP64;
  SortArgs a = sort_args(c, s, pred.tau, pred.a_mid);
  char* p = room.lists;
  auto list = [&](size_t words) { uint32_t* q = (uint32_t*)p; p += align_up(words * 4); return q; };
  a.count = list(a.nkeys);
  a.scan_scratch = list(sort_scan_scratch_words(a.nkeys));
  a.rank = list(s.n);
  a.bucket = list(s.n);
  a.src = list(s.n);
  launch_sort_rank(a, stream_of(c));
  // the state arrays by move-mask bit
  Segment& g = s.seg[0];
  void** home[10];
  for (int d = 0; d < 3; ++d) {
    home[d] = f64 ? (void**)&g.xd[d] : (void**)&g.xu[d];
    home[3 + d] = f64 ? (void**)&g.qd[d] : (void**)&g.q0f[d];
    home[6 + d] = f64 ? (void**)&g.q0d[d] : (void**)&g.dqf[d];
  }
  home[9] = (void**)&g.id;
  const bool resample = s.pristine;   // the ids alone; sampled again into the new order
  for (int k = resample ? 9 : 0; k < 10;) {
    Segment& t = a.dst;
    t = g;
    void** there[10];
    for (int d = 0; d < 3; ++d) {
      there[d] = f64 ? (void**)&t.xd[d] : (void**)&t.xu[d];
      there[3 + d] = f64 ? (void**)&t.qd[d] : (void**)&t.q0f[d];
      there[6 + d] = f64 ? (void**)&t.q0d[d] : (void**)&t.dqf[d];
    }
    there[9] = (void**)&t.id;
    CopyArgs cp{};
    size_t used = 0;
    a.move_mask = 0;
    for (; k < 10; ++k) {
      const size_t bytes = (size_t)s.n * (f64 && k < 9 ? 8 : 4);
      if (used + align_up(bytes) > room.array_bytes) break;
      *there[k] = room.arrays + used;
      used += align_up(bytes);
      a.move_mask |= 1u << k;
      cp.src[cp.n] = (const uint32_t*)*there[k];
      cp.dst[cp.n] = (uint32_t*)*home[k];
      cp.words[cp.n++] = (int64_t)(bytes / 4);
    }
    launch_sort_move(a, stream_of(c));
    launch_copy(cp, stream_of(c));
  }
  if (resample) launch_sample_species(resample_args(c, s, g), stream_of(c));
  return launched(c, "sort in place");
}

// Rank and move passes of one species into its other buffer copy (or in
// place).  resample: a species whose state is still the sampled one moves its
// ids alone and is sampled again, by id, into the sorted slots (the same
// values as moving the whole state from the random sampling order, at a
// fraction of the scattered writes).
int sort_species(fdf_ctx* c, SpeciesRec& s, const SortPrediction& pred, bool resample) {
  std::pair<hipEvent_t, hipEvent_t> ev;
  timing_begin(c, FDF_KERNEL_SORT, &ev);
  InPlaceRoom room;
  if (in_place_room(c, s.n, &room)) {
    const int rc = sort_in_place(c, s, pred, room);
    if (rc) return rc;
  } else {
    SortArgs a = sort_args(c, s, pred.tau, pred.a_mid);
    const bool ids = resample && s.pristine;
    a.move_mask = ids ? kMoveIds : kMoveAll;
    launch_sort(a, stream_of(c));
    if (ids) launch_sample_species(resample_args(c, s, s.seg[s.cur ^ 1]), stream_of(c));
    s.cur ^= 1;
  }
  timing_end(c, FDF_KERNEL_SORT, ev);
  return launched(c, "sort");
}

// The steps of one fdf_step call.  Launch index j in [0, n] stands for the
// kick at integer time time(j) and (j < n) the drift to time(j + 1).
struct StepPlan {
  const fdf_ctx* c;
  int k0, n;                 // first integer time and signed number of steps
  int nabs() const { return std::abs(n); }
  int time(int j) const { return n > 0 ? k0 + j : k0 - j; }
  // drift from integer time u in the direction of the call (false past the schedule's end)
  bool drift(int u, double* dr, double* ah) const {
    if (n > 0 ? u >= c->cfg.n_steps : u <= 0) return false;
    *dr = n > 0 ? c->drift[u] : -c->drift[u - 1];
    *ah = n > 0 ? c->a_half[u] : c->a_half[u - 1];
    return true;
  }
  PushStep step(int j) const {
    PushStep s{};
    const int t = time(j);
    double kclose = 0, kopen = 0;   // half-kicks ending / starting at t
    if (n > 0) {
      if (j > 0) kclose = c->kick2[t - 1];
      if (j < nabs()) kopen = c->kick1[t];
    } else {
      if (j > 0) kclose = -c->kick1[t];
      if (j < nabs()) kopen = -c->kick2[t - 1];
    }
    // the separable force does not depend on q: both halves as one kick
    const bool sep = c->cfg.eom == FDF_EOM_SEPARABLE;
    s.kick = sep ? kclose + kopen : kclose;
    s.kick_open = sep ? 0.0 : kopen;
    s.a_kick = c->a[t];
    s.do_drift = j < nabs();
    if (s.do_drift) drift(t, &s.drift, &s.a_drift);
    s.dscale = (float)(s.drift * 4294967296.0 / c->cfg.box_mpc);
    return s;
  }
};

// The re-sort cadence of a species at integer time u: whether it is due, and
// the steps until it is due next (from u; at least one).  Adaptive cadence:
// once its typical drift since order_time reaches sort_cells (and at the
// start); fixed cadence: at multiples of sort_every.
struct SortCadence {
  bool sorted;
  bool placed;
  int order_time;
  double drift_cells;
  int waited;                // its first order in place was left to a later call: kThisCall, kEarlierCall
  double cells;              // adaptive threshold (0: fixed cadence)
  int every;                 // fixed cadence (0: never)
  int first_order;           // gathers for which a first order is made (0: any number)
  SortCadence restart(int time) const { return SortCadence{true, false, time, 0.0, 0, cells, every, first_order}; }
};
constexpr int kNeverDue = 1 << 30;

// Looks `most` steps ahead at most and says kNeverDue beyond: a caller that only
// asks whether a launch's span reaches that far must not walk a long schedule to
// its end at every launch (20 000 steps, three species: 0.12 ms a call).
int steps_until_due(fdf_ctx* c, const StepPlan& p, const SortCadence& s, int u, double m, int most = kNeverDue) {
  const int dir = p.n > 0 ? 1 : -1;
  if (s.cells > 0) {
    double cells = s.drift_cells, dr, ah;
    for (int k = 1; k <= most && p.drift(u, &dr, &ah); ++k, u += dir) {
      cells += typical_drift_cells(c, dr, ah, m);
      if (cells >= s.cells) return k;
    }
    return kNeverDue;
  }
  if (s.every <= 0) return kNeverDue;
  const int r = u % s.every;
  return dir > 0 ? s.every - r : (r ? r : s.every);
}

// A species in the order of its creation is due at once if its particles will
// drift further than this (in cells) over the gathers of the first interval: a
// re-sort orders by the positions at the middle of the interval, creation by
// those at its start.
constexpr double kPlacedDrift = 3.0;

// A first order in place pays in a call of this many gathers: its cost, over
// what a gather gains by it.  Particles in a given order, 2 M on 128^3, us without
// and with it:  FP32 CIC, 6 gathers 697 and 684;  FP32 TSC, 2 684 and 707, 3 992
// and 765;  FP64 CIC, 4 1038 and 1052, 5 1294 and 1104;  FP64 TSC, 2 1584 and
// 1220.  Its launches take as long as its passes over 270 K particles: 200 K on
// 128^3, FP32 CIC, 6 gathers 100 and 157, 12 174 and 176.  Sparse particles share
// few mesh lines in any order: 300 K on 256^3, 12 gathers 362 and 445, FP64 TSC
// 1884 and 1806.  A first call of fewer leaves it to the second one, which more
// are likely to follow.
int first_order_gathers(const fdf_ctx* c, int64_t n) {
  const bool f64 = c->cfg.precision == FDF_PREC_FP64;
  const int64_t G = c->cfg.grid_n;
  if (32 * n < G * G * G) return kMaxSpan;
  const double large = c->cfg.interp_order == 2 ? (f64 ? 1.5 : 2.4) : (f64 ? 4.6 : 6.0);
  return (int)std::min<double>(kMaxSpan, std::lround(large * (1.0 + 270e3 / (double)n)));
}

enum class Due { kNo, kWaits, kNow };   // kWaits: for a later call

// gathers: those left in the call, from integer time u on.
Due sort_due(fdf_ctx* c, const StepPlan& p, const SortCadence& s, int u, double m, int gathers) {
  const Due first = gathers >= s.first_order || s.waited == kEarlierCall ? Due::kNow : Due::kWaits;
  if (s.cells > 0 && s.sorted && s.drift_cells >= s.cells) return Due::kNow;
  if (s.placed && (s.cells > 0 || s.every > 0)) {
    const int dir = p.n > 0 ? 1 : -1;
    const int len = s.cells > 0 ? kNeverDue : steps_until_due(c, p, s, u, m);
    double dr, ah, cells = 0.0;
    for (int k = 1; k < len && p.drift(u + dir * (k - 1), &dr, &ah); ++k) {
      cells += typical_drift_cells(c, dr, ah, m);
      if (s.cells > 0 && cells >= s.cells) break;   // the interval ends here
      if (cells > kPlacedDrift) return first;
    }
  }
  if (s.cells > 0) return s.sorted ? Due::kNo : first;
  return s.every > 0 && u % s.every == 0 && s.order_time != u ? Due::kNow : Due::kNo;
}

// Adaptive threshold of the re-sorts in place.  They cost two passes more than
// a re-sort into a second copy, so they wait longer: 16.8 M particles on 256^3,
// 40 steps, FP64 72, 63, 60 and 58 ms at 3, 6, 9 and 14 cells (102 ms without
// them), 2 M TSC 13.0, 12.8, 13.2 and 14.7 ms (22); FP32 23.7, 21.9 and 20.7 ms
// at 6, 9 and 14 cells (27 ms).
constexpr double kInPlaceCells = 10.0;

SortCadence cadence_of(fdf_ctx* c, const SpeciesRec& s) {
  SortCadence r{s.sorted, s.placed, s.order_time, s.drift_cells, s.waited, c->sort_cells, c->sort_every, 0};
  InPlaceRoom room;
  if (in_place_room(c, s.n, &room)) {
    r.cells = kInPlaceCells;
    r.first_order = first_order_gathers(c, s.n);
  }
  return r;
}

// Positions to order by for the interval that starts `lead` steps after u (as
// long as the cadence will let it be): the state at u extrapolated to the
// middle of the interval's gathers, which are made at the start of each of its
// steps.
SortPrediction sort_prediction(fdf_ctx* c, const StepPlan& p, const SortCadence& s, int u, int lead, double m) {
  const int dir = p.n > 0 ? 1 : -1, u0 = u + dir * lead;
  const int len = steps_until_due(c, p, s.restart(u0), u0, m);
  double dr, ah, before = 0.0, span = 0.0;
  for (int k = 0; k < lead && p.drift(u + dir * k, &dr, &ah); ++k) before += dr;
  for (int k = 0; k + 1 < len && p.drift(u0 + dir * k, &dr, &ah); ++k) span += dr;
  const double tau = before + 0.5 * span;
  // scale factor half way along the extrapolation
  SortPrediction r;
  r.a_mid = c->a[u];
  double done = 0.0;
  for (int v = u; p.drift(v, &dr, &ah); v += dir) {
    if (std::fabs(done) > 0.5 * std::fabs(tau)) break;
    r.a_mid = ah;
    done += dr;
  }
  r.tau = c->sort_predict ? tau : 0.0;
  return r;
}

// What the next launch does for a species standing at launch index j.
struct LaunchPlan {
  int span = 1;              // steps carried out
  bool waits = false;        // a first order in place is left to a later call
  bool sort_first = false;   // rank and move passes before it (sort_passes of them)
  int sort_passes = 0;
  bool fused = false;        // the push writes the state in sorted order for the interval after it
  SortPrediction pred;       // of the rank pass before a fused push
  SortPrediction pred_first; // of the rank and move passes
};

// limit: launch indices [j, limit) see the same grids.
LaunchPlan plan_launch(fdf_ctx* c, const StepPlan& p, const SortCadence& s, double m, int j, int limit) {
  LaunchPlan l;
  const int u = p.time(j), rem = p.nabs() - j;   // drift steps left in the call
  const int room = std::min(limit - j, kMaxSpan);
  if (rem == 0) return l;                         // the closing kick
  const int dir = p.n > 0 ? 1 : -1;
  const bool fusable = c->cfg.sort_every > 0 && c->sort_fused && c->cfg.precision == FDF_PREC_FP32 &&
                       c->cfg.eom == FDF_EOM_SEPARABLE;
  double dr, ah;
  SortCadence now = s;
  const Due due = sort_due(c, p, s, u, m, rem + 1);
  l.waits = due == Due::kWaits;
  if (due == Due::kNow) {
    // a first sort takes two passes (the second orders cells in buckets)
    const bool first = !s.sorted;
    const bool ride = fusable && p.drift(u + dir, &dr, &ah);   // steps follow that use the new order
    l.sort_passes = (first ? 2 : 1) - (ride ? 1 : 0);
    l.sort_first = l.sort_passes > 0;
    if (l.sort_first) l.pred_first = sort_prediction(c, p, s, u, 0, m);
    if (ride) {
      l.fused = true;
      l.pred = sort_prediction(c, p, s, u, 1, m);
      return l;
    }
    now = s.restart(u);
  }
  const int d = l.waits && !s.sorted ? kNeverDue : steps_until_due(c, p, now, u, m, room);
  if (d < rem) {               // due again within the call
    l.span = std::min(d, room);
    if (fusable && l.span == d) {
      l.fused = true;
      l.pred = sort_prediction(c, p, s, u, d, m);
    }
  } else {
    l.span = std::min(rem + 1, room);   // to the end of the call, the closing kick included
  }
  return l;
}

// The species' cadence after the launch.
SortCadence after_launch(fdf_ctx* c, const StepPlan& p, const SortCadence& s, const LaunchPlan& l, double m, int j) {
  const int dir = p.n > 0 ? 1 : -1, u = p.time(j);
  SortCadence r = s;
  r.placed = s.placed && (l.waits || j == p.nabs());   // (or a closing kick on its own)
  if (l.waits) r.waited = kThisCall;
  if (l.sort_first) r = s.restart(u);
  double dr, ah;
  for (int k = 0; k < l.span && j + k < p.nabs(); ++k)
    if (p.drift(u + dir * k, &dr, &ah)) r.drift_cells += typical_drift_cells(c, dr, ah, m);
  if (l.fused) r = s.restart(u + dir * l.span);
  return r;
}

// One species of a launch: what it does there, and the rank pass after it
// for which the launch writes the sort keys.
struct LaunchMember {
  size_t species = 0;
  LaunchPlan plan;
  bool keyed = false;        // the species' previous push has written its sort keys
  bool writes_keys = false;
  SortPrediction next;
};

// A launch that would have fewer than this many blocks takes fewer particles
// per thread: 256 CUs need several blocks each to hide their gathers (64^3
// particles, 24 steps: 75 us with 256 blocks of 4 per thread, 46 us with 1024
// of 1 per thread).
constexpr int64_t kMinPushBlocks = 2048;
// LDS reserved per block of a wide or re-sorting push so that a CU holds one
// block of 1024 particles.  Over several steps the gathers are bound by the
// address unit and the 32 KB L1, whose hits come from particles that are
// neighbours in the order: 1024 of them touch about 33 KB of a bfloat16 mesh,
// and a second block on the CU, from elsewhere in the order, evicts it.
// 512^3 particles, 6.4 steps per re-sorting launch: 9.73, 9.42 and 9.10 ms with
// 1, 2 and 4 particles per thread and as many blocks as fit, 8.77, 9.21 and
// 13.1 ms with one block; one step: 4.16 -> 4.09 ms with 1 per thread;
// super-steps on 256^3: 2.89 -> 2.30 ms.  Sparse species
// (below half a particle per mesh cell) touch more lines per particle and want
// fewer waves: 100 M on 13 meshes of 256^3, 6.36 ms with 2 per thread, 6.7 with 1.
constexpr int kOneBlockReserve = 90 * 1024;
// Super-steps with TSC on 8 slots above 4 GiB of mesh (64-bit gather addresses):
// with one particle per thread, 1024 threads of it, the re-sorting push keeps 44
// registers in memory.  560 M particles on 1024^3, 5 launches: 1077, 614 and 560
// ms with 1, 2 and 4 per thread; 60 M (sparse) 221 ms with 2, 173 with 4.  Below
// 4 GiB the same kernel keeps 2 there: 60 M on 256^3 130, 131 and 141 ms.
bool wide_blended_gather(const PushArgs& a) {
  return a.blend && a.tsc && a.nslot == 8 && (uint64_t)a.G * a.G * a.G * 16 > (1ull << 32);
}

// One launch over the members (at most kMaxJobs), all standing at the same
// launch index (pa.step[0]) and all fused or all plain.
int run_launch(fdf_ctx* c, PushArgs& pa, const std::vector<LaunchMember>& members) {
  const size_t table = align_up((size_t)c->cfg.max_species * sizeof(Segment));
  const bool fused = members[0].plan.fused;
  SpeciesBatch& b = pa.batch;
  b = SpeciesBatch{};
  b.tables[0] = (const Segment*)(c->ws + c->lay.seg);
  b.tables[1] = (const Segment*)(c->ws + c->lay.seg + table);
  int64_t total = 0;
  for (auto& m : members) total += c->species[m.species].n;
  int longest = 1;
  for (auto& m : members) longest = std::max(longest, m.plan.span);
  const bool one_each = pa.fp64 || pa.eom != FDF_EOM_SEPARABLE;   // kernels of one particle per thread
  // wide blocks: for launches of several steps that can give every CU one
  const bool wide = longest > 1 && !pa.tsc && pa.eom == FDF_EOM_SEPARABLE && total >= 256 * kPushWideBlock;
  std::vector<char> mesh(c->fields.size(), 0);
  for (auto& m : members) mesh[c->species[m.species].field] = 1;
  int64_t meshes = 0;
  for (char r : mesh) meshes += r;
  const int64_t cells = meshes * (int64_t)c->cfg.grid_n * c->cfg.grid_n * c->cfg.grid_n;
  if (fused) {
    pa.ppt = longest == 1 ? c->sort_push_ppt : wide_blended_gather(pa) ? 4 : 2 * total < cells ? 2 : 1;
  } else {
    pa.block = wide ? kPushWideBlock : kPushBlock;
    pa.ppt = wide || one_each ? 1 : c->ppt;
    pa.lds_reserve = wide ? kOneBlockReserve : push_lds_reserve(c->push_waves);
  }
  while (pa.ppt > 1 && total < kMinPushBlocks * kPushBlock * pa.ppt) pa.ppt /= 2;
  if (fused) pa.lds_reserve = pa.ppt <= 2 || (longest > 1 && wide_blended_gather(pa)) ? kOneBlockReserve : 0;
  const int64_t per = fused ? kSortBlock : pa.block * pa.ppt;
  const SortArgs sa = sort_args(c, c->species[members[0].species], 0.0, 0.0);
  pa.key_out = (uint32_t*)(c->ws + c->lay.sort_key);
  pa.key_mask = 0;
  pa.key_fine_bits = sa.fine_bits;
  int64_t blocks = 0, base = 0;
  for (auto& m : members) {
    const SpeciesRec& s = c->species[m.species];
    const int j = b.njobs++;
    b.job_species[j] = (int32_t)m.species;
    b.job_cur[j] = s.cur;
    b.job_block[j] = blocks;
    b.job_base[j] = base;
    for (size_t i = 0; i < m.species; ++i) b.job_slot[j] += c->species[i].n;
    b.job_tau[j] = m.plan.pred.tau;
    b.job_ma[j] = s.m * m.plan.pred.a_mid;
    if (m.keyed) b.keyed_mask |= 1u << j;
    if (m.writes_keys) pa.key_mask |= 1u << j;
    pa.key_tau[j] = m.next.tau;
    pa.key_ma[j] = s.m * m.next.a_mid;
    pa.nsteps[j] = (int8_t)m.plan.span;
    blocks += (s.n + per - 1) / per;
    base += s.n;
  }
  b.job_block[b.njobs] = blocks;
  pa.grid_blocks = batch_grid(b);
  std::pair<hipEvent_t, hipEvent_t> ev;
  const int cls = fused ? FDF_KERNEL_PUSH_SORT : FDF_KERNEL_PUSH;
  if (fused) {
    SortArgs a = sa;
    a.batch = b;
    a.keys = (const uint32_t*)(c->ws + c->lay.sort_key);
    timing_begin(c, FDF_KERNEL_SORT, &ev);
    launch_sort_rank_batch(a, stream_of(c));
    timing_end(c, FDF_KERNEL_SORT, ev);
    pa.sort_src = a.src;
    pa.sort_rank = a.rank;
    pa.sort_bucket = a.bucket;
    pa.sort_start = a.count;
    pa.sort_nkeys = a.nkeys;
    timing_begin(c, cls, &ev);
    launch_push_sort(pa, stream_of(c));
    timing_end(c, cls, ev);
  } else {
    timing_begin(c, cls, &ev);
    launch_push(pa, stream_of(c));
    timing_end(c, cls, ev);
  }
  timing_work(c, cls, 0, pa.step, 0, cells * (pa.blend ? 2 : 1));
  for (auto& m : members) {
    SpeciesRec& s = c->species[m.species];
    timing_work(c, cls, s.n, pa.step, m.plan.span, 0);
    if (fused) s.cur ^= 1;
    s.pristine = false;
  }
  return launched(c, fused ? "sort + push" : "push");
}

OutputArgs output_args(fdf_ctx* c, const SpeciesRec& s) {
  OutputArgs o{};
  o.seg = s.seg[s.cur];
  o.fp64 = c->cfg.precision == FDF_PREC_FP64;
  o.G = c->cfg.grid_n;
  o.pre_ic = (s.flags & FDF_SPECIES_PRE_IC) != 0;
  o.seed = s.seed;
  o.t_nu = t_nu_ev();
  o.box = c->cfg.box_mpc;
  o.a = c->a[c->step_index];
  o.m = s.m;
  return o;
}

// First complex entry of the n-point table in the twiddle regions.
size_t twiddle_entry(int G, int n) { return 2 * (size_t)(G - n); }

void fill_twiddles(fdf_ctx* c) {
  const int G = c->cfg.grid_n;
  std::vector<double> td(4 * (size_t)G, 0.0);
  std::vector<float> tf(4 * (size_t)G, 0.0f);
  for (int n = G; n >= 8; n /= 2) {
    const size_t base = 2 * twiddle_entry(G, n);
    for (int m = 0; m < n; ++m) {
      const long double ang = -2.0L * 3.141592653589793238462643383279502884L * m / n;
      td[base + 2 * m] = (double)cosl(ang);
      td[base + 2 * m + 1] = (double)sinl(ang);
      tf[base + 2 * m] = (float)cosl(ang);
      tf[base + 2 * m + 1] = (float)sinl(ang);
    }
  }
  (void)hipMemcpy(c->ws + c->lay.twiddle_d, td.data(), td.size() * 8, hipMemcpyHostToDevice);
  (void)hipMemcpy(c->ws + c->lay.twiddle_f, tf.data(), tf.size() * 4, hipMemcpyHostToDevice);
}

int add_field_slot(fdf_ctx* c, int32_t* id) {
  if ((int)c->fields.size() >= c->cfg.max_fields) return fail(c, FDF_ERR_CAPACITY, "max_fields reached");
  FieldRec f;
  char* base = c->ws + c->lay.fields + c->field_next;
  f.dk = base;
  f.grid = base + c->lay.field_dk_bytes;
  f.grid2 = c->lay.grid_sets > 1 ? base + c->lay.field_dk_bytes + c->lay.field_grid_bytes : nullptr;
  c->field_next += c->lay.field_dk_bytes + c->lay.grid_sets * c->lay.field_grid_bytes;
  c->fields.push_back(f);
  *id = (int32_t)c->fields.size() - 1;
  return FDF_OK;
}

int new_species(fdf_ctx* c, int32_t field_id, double m, int64_t n, uint64_t seed, int flags, int32_t* sid) {
  if (field_id < 0 || field_id >= (int)c->fields.size()) return fail(c, FDF_ERR_ARG, "bad field id");
  if (!(m >= 0) || !std::isfinite(m)) return fail(c, FDF_ERR_ARG, "mass must be finite and >= 0");
  if (n < 1) return fail(c, FDF_ERR_ARG, "need at least one particle");
  if (c->stepped) return fail(c, FDF_ERR_STATE, "species must be added before the first step");
  if ((int)c->species.size() >= c->cfg.max_species) return fail(c, FDF_ERR_CAPACITY, "max_species reached");
  int64_t tot = n;
  for (auto& s : c->species) tot += s.n;
  if (tot > c->cfg.max_particles) return fail(c, FDF_ERR_CAPACITY, "max_particles exceeded");
  SpeciesRec s;
  s.field = field_id; s.m = m; s.n = n; s.seed = seed; s.flags = flags;
  const size_t save = c->part_next;
  if (!carve_species(c, s.seg[0], n)) { c->part_next = save; return fail(c, FDF_ERR_CAPACITY, "workspace particles full"); }
  if (c->cfg.sort_every > 0 && !carve_species(c, s.seg[1], n)) {
    c->part_next = save;
    return fail(c, FDF_ERR_CAPACITY, "workspace particles full");
  }
  c->species.push_back(s);
  c->seg_dirty = true;
  *sid = (int32_t)c->species.size() - 1;
  return FDF_OK;
}

// Puts the ids of a new species in the spatial order of its sampled positions
// (its state is then sampled by id).  Every gather and deposit runs on that
// order until the particles have drifted out of it, which a context that
// never re-sorts has no other way to get, and it stands in for a first sort.
// Not done for a mesh that one XCD's L2 holds in a context without re-sorts
// (the gathers hit there in any order), when the temporaries (8 B per
// particle and the tile counts, in the sort's arrays or else in the FFT
// scratch) do not fit, or when they would overwrite a density that can still
// be read.  Returns whether the ids are in order.
bool place_species(fdf_ctx* c, SpeciesRec& s) {
  const int G = c->cfg.grid_n, tiles = std::min(G, 256);
  const bool sorting = c->cfg.sort_every > 0;
  if (!sorting && (c->lay.field_grid_bytes <= kL2Bytes || c->have_density)) return false;
  PlaceArgs a{};
  a.seg = s.seg[0];
  a.seed = s.seed;
  a.cell_shift = 32 - ilog2(G);
  a.fine_bits = ilog2(G / tiles);
  a.nkeys = (int64_t)tiles * tiles * tiles;
  if (sorting) {
    a.count = (uint32_t*)(c->ws + c->lay.sort_count);
    a.scan_scratch = (uint32_t*)(c->ws + c->lay.sort_scan);
    a.key = (uint32_t*)(c->ws + c->lay.sort_bucket);
    a.binned = (uint32_t*)(c->ws + c->lay.sort_rank);
  } else {
    // the FFT scratch and the density halves behind it
    const size_t count = align_up((size_t)a.nkeys * 4), scan = align_up(sort_scan_scratch_words(a.nkeys) * 4);
    const size_t list = align_up((size_t)s.n * 4);
    if (count + scan + 2 * list > c->lay.scratch_bytes + c->lay.dens_bytes) return false;
    char* p = c->ws + c->lay.scratch;
    a.count = (uint32_t*)p;
    a.scan_scratch = (uint32_t*)(p + count);
    a.key = (uint32_t*)(p + count + scan);
    a.binned = (uint32_t*)(p + count + scan + list);
  }
  launch_place_species(a, c->stream);
  return true;
}

}  // namespace

// -------------------------------------------- static scratch (no allocation) --
// Device memory of fdf_power_spectrum_noalloc: one array per GPU, held until
// the process ends.  Host code never passes `scratch` itself to a kernel or a
// copy; it uses the address hipGetSymbolAddress returns for the current device.
constexpr size_t kStaticScratchBytes = (size_t)16 << 20;
constexpr int kStaticMaxMesh = 64;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {};

// The static scratch of the current device (resolved once per device).
int static_scratch(fdf_ctx* c, char** out) {
  int dev = -1;
  int rc = hip_check(c, hipGetDevice(&dev), "hipGetDevice");
  if (rc) return rc;
  if (dev < 0 || dev >= kMaxDevices) return fail(c, FDF_ERR_UNSUPPORTED, "device index beyond the static scratch table");
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    rc = hip_check(c, hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)), "hipGetSymbolAddress(scratch)");
    if (rc) return rc;
    g_scratch_ptr[dev] = ptr;
  }
  *out = (char*)g_scratch_ptr[dev];
  return FDF_OK;
}

// Static scratch bytes of a spectrum on a G^3 mesh: bins, the maximum word,
// the deposit halves (8 bytes per cell each), four FFT planes and (FP32 form)
// the binary32 halves.
size_t static_scratch_bytes(bool f64, int G) {
  const size_t g3 = (size_t)G * G * G, plane = (size_t)G * G * (G / 2) * (f64 ? 16 : 8);
  return align_up(kBinsBytes) + kAlign + align_up(2 * g3 * 8) + align_up(4 * plane) +
         (f64 ? 0 : align_up(2 * g3 * 4));
}

}  // namespace

// ============================================================== C ABI ======
extern "C" {

const char* fdf_status_string(int s) {
  switch (s) {
    case FDF_OK: return "ok";
    case FDF_ERR_ARG: return "invalid argument";
    case FDF_ERR_STATE: return "invalid state";
    case FDF_ERR_WORKSPACE: return "workspace missing or too small";
    case FDF_ERR_HIP: return "HIP runtime error";
    case FDF_ERR_CAPACITY: return "capacity exceeded";
    case FDF_ERR_UNSUPPORTED: return "unsupported";
    default: return "unknown status";
  }
}

const char* fdf_last_error(const fdf_ctx* c) { return c ? c->err.c_str() : "null context"; }

int fdf_workspace_size(const fdf_config* cfg, size_t* bytes) {
  if (validate(cfg) || !bytes) return FDF_ERR_ARG;
  *bytes = plan(*cfg).total;
  return FDF_OK;
}

int fdf_create(const fdf_config* cfg, void* stream, fdf_ctx** out) {
  if (!out) return FDF_ERR_ARG;
  *out = nullptr;
  if (validate(cfg)) return FDF_ERR_ARG;
  fdf_ctx* c = new fdf_ctx();
  c->cfg = *cfg;
  c->cos = Cosmo{cfg->h, cfg->omega_m, cfg->omega_r, cfg->omega_l};
  c->stream = (hipStream_t)stream;
  c->lay = plan(*cfg);
  const int n = cfg->n_steps;
  const double lai = std::log(1.0 / (1.0 + cfg->z_begin)), laf = std::log(1.0 / (1.0 + cfg->z_end));
  const double dl = (laf - lai) / n;
  c->a.resize(n + 1);
  c->a_half.resize(n);
  c->kick1.resize(n);
  c->kick2.resize(n);
  c->drift.resize(n);
  for (int k = 0; k <= n; ++k) c->a[k] = std::exp(lai + dl * k);
  double max_drift = 0;
  for (int k = 0; k < n; ++k) {
    const double l0 = lai + dl * k, lh = lai + dl * (k + 0.5), l1 = lai + dl * (k + 1);
    c->a_half[k] = std::exp(lh);
    c->kick1[k] = dtau(c->cos, l0, lh);
    c->kick2[k] = dtau(c->cos, lh, l1);
    c->drift[k] = dtau(c->cos, l0, l1);
    max_drift = std::max(max_drift, std::fabs(c->drift[k]));
  }
  if (!(max_drift < 0.5 * cfg->box_mpc)) {   // fixed-point drift must stay below half a box
    delete c;
    return FDF_ERR_ARG;
  }
  c->amp = power_amplitude(cfg->sigma8, cfg->ns, cfg->gamma, cfg->h);
  c->sort_every = cfg->sort_every;
  if (cfg->potential_model == FDF_MODEL_RADMAT && cfg->superstep_tol > 0) {
    // Super-steps (sec. 2.1): a new anchor where phi or psi changed by more
    // than the tolerance since the last one (the model's transfer functions
    // are k-independent multiples of g(a), so the ratio test uses g alone).
    double g0, dg0, g, dg;
    radmat_factor(c->a[0], cfg->omega_m, cfg->omega_r, &g0, &dg0);
    c->anchors.push_back(0);
    for (int k = 1; k <= n; ++k) {
      radmat_factor(c->a[k], cfg->omega_m, cfg->omega_r, &g, &dg);
      if (std::fabs(g / g0 - 1.0) > cfg->superstep_tol) {
        c->anchors.push_back(k);
        g0 = g;
      }
    }
    if (c->anchors.back() != n) c->anchors.push_back(n);
  }
  c->tau_begin = conformal_time(c->cos, c->a[0]);
  *out = c;
  return FDF_OK;
}

int fdf_attach_workspace(fdf_ctx* c, void* dptr, size_t bytes) {
  if (!c) return FDF_ERR_ARG;
  if (!dptr || ((uintptr_t)dptr % kAlign) != 0) return fail(c, FDF_ERR_WORKSPACE, "workspace must be 256-byte aligned");
  if (bytes < c->lay.total) return fail(c, FDF_ERR_WORKSPACE, "workspace too small");
  clear_graphs(c);   // captured launches hold addresses of the workspace before
  c->ws = (char*)dptr;
  c->ws_bytes = bytes;
  fill_twiddles(c);
  char* st = nullptr;
  int rc = static_scratch(c, &st);   // set-up of the no-allocation entry point's scratch
  if (!rc && !c->pinned)
    rc = hip_check(c, hipHostMalloc((void**)&c->pinned, 3 * kMaxBins * sizeof(double)), "page-locked bins");
  if (rc) return rc;
  return fdf_reset(c);
}

int fdf_reset(fdf_ctx* c) {
  if (!c) return FDF_ERR_ARG;
  c->fields.clear();
  c->species.clear();
  c->field_next = 0;
  c->part_next = 0;
  c->step_index = 0;
  c->stepped = false;
  c->seg_dirty = true;
  c->have_density = false;
  return FDF_OK;
}

int fdf_destroy(fdf_ctx* c) {
  if (!c) return FDF_ERR_ARG;
  (void)hipStreamSynchronize(c->stream);
  clear_graphs(c);
  if (c->cap_stream) (void)hipStreamDestroy(c->cap_stream);
  if (c->pinned) (void)hipHostFree(c->pinned);
  for (auto& t : c->tim) {
    for (auto& e : t.pending) { (void)hipEventDestroy(e.first); (void)hipEventDestroy(e.second); }
    for (auto& e : t.pool) { (void)hipEventDestroy(e.first); (void)hipEventDestroy(e.second); }
  }
  delete c;
  return FDF_OK;
}

int fdf_add_field(fdf_ctx* c, uint64_t seed, int32_t fixed_amp, int32_t* field_id) {
  if (!c || !field_id) return FDF_ERR_ARG;
  if (!needs_ws(c)) return fail(c, FDF_ERR_WORKSPACE, "no workspace attached");
  int rc = add_field_slot(c, field_id);
  if (rc) return rc;
  FieldRec& f = c->fields.back();
  f.seed = seed;
  FieldGenArgs g{};
  g.G = c->cfg.grid_n;
  g.fp64 = c->cfg.precision == FDF_PREC_FP64;
  g.fixed_amp = fixed_amp;
  g.seed = seed;
  g.box = c->cfg.box_mpc;
  g.amp = c->amp;
  g.ns = c->cfg.ns;
  g.gamma = c->cfg.gamma;
  g.h = c->cfg.h;
  g.out = f.dk;
  std::pair<hipEvent_t, hipEvent_t> ev;
  timing_begin(c, FDF_KERNEL_INIT, &ev);
  launch_field_gen(g, c->stream);
  timing_end(c, FDF_KERNEL_INIT, ev);
  return launched(c, "field generation");
}

int fdf_set_field(fdf_ctx* c, const double* h, int32_t* field_id) {
  if (!c || !h || !field_id) return FDF_ERR_ARG;
  if (!needs_ws(c)) return fail(c, FDF_ERR_WORKSPACE, "no workspace attached");
  int rc = add_field_slot(c, field_id);
  if (rc) return rc;
  const int G = c->cfg.grid_n, M = G / 2, H = G / 2 + 1;
  const bool f64 = c->cfg.precision == FDF_PREC_FP64;
  std::vector<double> d((size_t)G * G * M * 2);
  std::vector<float> f(f64 ? 0 : d.size());
  for (int ix = 0; ix < G; ++ix)
    for (int iy = 0; iy < G; ++iy)
      for (int iz = 0; iz < M; ++iz) {
        const size_t src = (((size_t)ix * G + iy) * H + iz) * 2, dst = (((size_t)ix * G + iy) * M + iz) * 2;
        const bool nyq = ix == M || iy == M;
        d[dst] = nyq ? 0.0 : h[src];
        d[dst + 1] = nyq ? 0.0 : h[src + 1];
      }
  if (!f64) for (size_t i = 0; i < d.size(); ++i) f[i] = (float)d[i];
  rc = hip_check(c, hipMemcpyAsync(c->fields.back().dk, f64 ? (void*)d.data() : (void*)f.data(),
                                   d.size() * (f64 ? 8 : 4), hipMemcpyHostToDevice, c->stream), "field upload");
  if (rc) return rc;
  return hip_check(c, hipStreamSynchronize(c->stream), "field upload");
}

int fdf_init_species(fdf_ctx* c, int32_t field_id, double m, int64_t n, uint64_t seed, int32_t flags,
                     int32_t* species_id) {
  if (!c || !species_id) return FDF_ERR_ARG;
  if (!needs_ws(c)) return fail(c, FDF_ERR_WORKSPACE, "no workspace attached");
  if (flags & ~FDF_SPECIES_PRE_IC) return fail(c, FDF_ERR_ARG, "unknown species flag");
  int rc = new_species(c, field_id, m, n, seed, flags, species_id);
  if (rc) return rc;
  SpeciesRec& s = c->species.back();
  SampleArgs sa{};
  sa.seg = s.seg[0];
  sa.fp64 = c->cfg.precision == FDF_PREC_FP64;
  sa.seed = seed;
  sa.box = c->cfg.box_mpc;
  sa.t_nu = t_nu_ev();
  std::pair<hipEvent_t, hipEvent_t> ev;
  timing_begin(c, FDF_KERNEL_INIT, &ev);
  if (place_species(c, s)) {
    sa.by_id = 1;
    s.sorted = s.placed = true;
    s.order_time = c->step_index;
  }
  launch_sample_species(sa, c->stream);
  if (flags & FDF_SPECIES_PRE_IC) {
    c->have_density = false;
    GridBuildArgs g = grid_recipe(c, c->fields[field_id], c->a[0], true);
    launch_build_grids(g, c->stream);
    PreIcArgs p{};
    p.seg = s.seg[0];
    p.fp64 = sa.fp64;
    p.G = c->cfg.grid_n;
    p.box = c->cfg.box_mpc;
    p.m = m;
    p.a = c->a[0];
    p.tau = c->tau_begin;
    p.grid = g.out;
    launch_pre_ic(p, c->stream);
  }
  timing_end(c, FDF_KERNEL_INIT, ev);
  s.pristine = !(flags & FDF_SPECIES_PRE_IC);
  return launched(c, "species sampling");
}

int fdf_set_species_state(fdf_ctx* c, int32_t field_id, double m, int64_t n, const uint32_t* xu,
                          const float* q, int32_t* species_id) {
  if (!c || !xu || !q || !species_id) return FDF_ERR_ARG;
  if (!needs_ws(c)) return fail(c, FDF_ERR_WORKSPACE, "no workspace attached");
  int rc = new_species(c, field_id, m, n, 0, 0, species_id);
  if (rc) return rc;
  Segment& s = c->species.back().seg[0];
  const bool f64 = c->cfg.precision == FDF_PREC_FP64;
  std::vector<uint32_t> ids(n);
  for (int64_t i = 0; i < n; ++i) ids[i] = (uint32_t)i;
  std::vector<double> dd(f64 ? n : 0);
  std::vector<float> ff(f64 ? 0 : n), zero(f64 ? 0 : n, 0.0f);
  std::vector<uint32_t> uu(f64 ? 0 : n);
  auto put = [&](void* dst, const void* src, size_t bytes) {
    return hip_check(c, hipMemcpy(dst, src, bytes, hipMemcpyHostToDevice), "state upload");
  };
  for (int d = 0; d < 3 && !rc; ++d) {
    if (f64) {
      for (int64_t i = 0; i < n; ++i) dd[i] = (double)xu[3 * i + d] * (c->cfg.box_mpc * 0x1p-32);
      rc = put(s.xd[d], dd.data(), n * 8);
      for (int64_t i = 0; i < n; ++i) dd[i] = (double)q[3 * i + d];
      if (!rc) rc = put(s.qd[d], dd.data(), n * 8);
      if (!rc) rc = put(s.q0d[d], dd.data(), n * 8);
    } else {
      for (int64_t i = 0; i < n; ++i) { uu[i] = xu[3 * i + d]; ff[i] = q[3 * i + d]; }
      rc = put(s.xu[d], uu.data(), n * 4);
      if (!rc) rc = put(s.q0f[d], ff.data(), n * 4);
      if (!rc) rc = put(s.dqf[d], zero.data(), n * 4);
    }
  }
  if (!rc) rc = put(s.id, ids.data(), n * 4);
  return rc;
}

int fdf_build_potential_grids(fdf_ctx* c, int32_t field_id, double a) {
  if (!c) return FDF_ERR_ARG;
  if (!needs_ws(c)) return fail(c, FDF_ERR_WORKSPACE, "no workspace attached");
  if (field_id < 0 || field_id >= (int)c->fields.size()) return fail(c, FDF_ERR_ARG, "bad field id");
  if (!(a > 0) || !std::isfinite(a)) return fail(c, FDF_ERR_ARG, "a must be positive");
  c->fields[field_id].tag[0] = -1;   // buffer 0 no longer holds a super-step anchor
  return build_grid(c, field_id, a);   // graphs are keyed on grid_a, so replays stay consistent
}

}  // extern "C"

namespace {

// Enqueue the launches of n steps (grid rebuilds, re-sorts, pushes) on the
// current launch stream and advance the host-side state.  Particles are
// independent given the grids, so a launch carries a species through every
// step up to its next re-sort, the next change of the grids, the end of the
// call or kMaxSpan steps with its state in registers, and species with
// different cadences advance in launches of their own.
int enqueue_steps(fdf_ctx* c, int32_t n) {
  const StepPlan plan{c, c->step_index, n};
  const int nabs = plan.nabs();
  const bool tdep = c->cfg.potential_model == FDF_MODEL_RADMAT;
  int rc = FDF_OK;
  std::vector<int> used(c->fields.size(), 0);
  for (auto& s : c->species) {
    used[s.field] = 1;
    if (s.waited) s.waited = kEarlierCall;
  }
  PushArgs pa{};
  pa.fp64 = c->cfg.precision == FDF_PREC_FP64;
  pa.nslot = c->lay.nslot;
  pa.G = c->cfg.grid_n;
  pa.log2g = ilog2(c->cfg.grid_n);
  pa.box = c->cfg.box_mpc;
  pa.persistent = c->persistent;
  pa.eom = c->cfg.eom;
  pa.tsc = c->cfg.interp_order == 2;
  const size_t ns = c->species.size();
  const int tiles = sort_tiles_of(c);
  const int64_t sort_jobs = std::min<int64_t>(kMaxJobs, std::max<int64_t>(1, c->lay.sort_keys_max /
                                                                                ((int64_t)tiles * tiles * tiles)));
  std::vector<int> at(ns, 0);          // launch index each species stands at
  std::vector<char> keyed(ns, 0);      // its sort keys are written
  // anchors of the super-step interval that holds integer time t
  auto anchor_interval = [&](int t) {
    const auto& an = c->anchors;
    size_t iv = 0;
    while (iv + 2 < an.size() && an[iv + 1] <= t) ++iv;
    return iv;
  };
  // end of the launch indices from j on that see the same grids
  auto same_grids_end = [&](int j) {
    if (!tdep) return nabs + 1;
    int e = j + 1;
    if (!c->anchors.empty()) {
      const size_t iv = anchor_interval(plan.time(j));
      while (e <= nabs && anchor_interval(plan.time(e)) == iv) ++e;
    }
    return e;
  };
  for (int j0 = 0; j0 <= nabs;) {
    const int j1 = same_grids_end(j0);
    pa.blend = 0;
    int kA = 0, kB = 0;
    if (!c->anchors.empty()) {
      // super-steps: grids at the anchors around t, interpolated linearly in a
      const size_t iv = anchor_interval(plan.time(j0));
      kA = c->anchors[iv];
      kB = c->anchors[iv + 1];
      int fsel_all = -1;
      for (size_t f = 0; f < c->fields.size(); ++f) {
        if (!used[f]) continue;
        FieldRec& fr = c->fields[f];
        int fsel;
        if (fr.tag[0] == kA && fr.tag[1] == kB) fsel = 0;
        else if (fr.tag[1] == kA && fr.tag[0] == kB) fsel = 1;
        else if (fr.tag[0] == kA) { rc = build_grid(c, (int)f, c->a[kB], 1); fr.tag[1] = kB; fsel = 0; }
        else if (fr.tag[1] == kA) { rc = build_grid(c, (int)f, c->a[kB], 0); fr.tag[0] = kB; fsel = 1; }
        else if (fr.tag[0] == kB) { rc = build_grid(c, (int)f, c->a[kA], 1); fr.tag[1] = kA; fsel = 1; }
        else if (fr.tag[1] == kB) { rc = build_grid(c, (int)f, c->a[kA], 0); fr.tag[0] = kA; fsel = 0; }
        else {
          rc = build_grid(c, (int)f, c->a[kA], 0);
          if (!rc) rc = build_grid(c, (int)f, c->a[kB], 1);
          fr.tag[0] = kA;
          fr.tag[1] = kB;
          fsel = 0;
        }
        if (rc) return rc;
        if (fsel_all >= 0 && fsel != fsel_all) return fail(c, FDF_ERR_STATE, "grid sets of fields out of step");
        fsel_all = fsel;
      }
      pa.blend = 1;
      pa.grid_sel = fsel_all < 0 ? 0 : fsel_all;
    } else {
      const double a_kick = c->a[plan.time(j0)];
      for (size_t f = 0; f < c->fields.size(); ++f) {
        if (!used[f]) continue;
        if (!c->fields[f].has_grid || (tdep && c->fields[f].grid_a != a_kick)) {
          rc = build_grid(c, (int)f, a_kick);
          if (rc) return rc;
        }
      }
    }
    while (true) {
      // the species furthest behind share a launch, with steps of their own each
      int j = j1;
      for (size_t i = 0; i < ns; ++i) j = std::min(j, at[i]);
      if (j >= j1) break;
      std::vector<LaunchMember> members;
      int longest = 0;
      for (size_t i = 0; i < ns; ++i) {
        if (at[i] != j) continue;
        SpeciesRec& s = c->species[i];
        const SortCadence cad = cadence_of(c, s);
        LaunchMember m;
        m.species = i;
        m.plan = plan_launch(c, plan, cad, s.m, j, j1);
        if (!members.empty() && m.plan.fused != members[0].plan.fused) continue;
        if (members.size() >= (size_t)(m.plan.fused ? sort_jobs : kMaxJobs)) break;
        const SortCadence after = after_launch(c, plan, cad, m.plan, s.m, j);
        const int jn = j + m.plan.span;
        if (c->sort_keys_push && jn < nabs && !pa.fp64 && pa.eom == FDF_EOM_SEPARABLE) {
          const LaunchPlan ln = plan_launch(c, plan, after, s.m, jn, jn < j1 ? j1 : same_grids_end(jn));
          m.writes_keys = ln.fused && !ln.sort_first;
          m.next = ln.pred;
        }
        m.keyed = m.plan.fused && !m.plan.sort_first && keyed[i];
        for (int pass = 0; pass < m.plan.sort_passes; ++pass) {
          rc = sort_species(c, s, m.plan.pred_first, pass == 0);
          if (rc) return rc;
        }
        s.sorted = after.sorted;
        s.placed = after.placed;
        s.order_time = after.order_time;
        s.drift_cells = after.drift_cells;
        s.waited = after.waited;
        keyed[i] = m.writes_keys;
        at[i] = jn;
        longest = std::max(longest, m.plan.span);
        members.push_back(m);
      }
      for (int k = 0; k < longest; ++k) {
        pa.step[k] = plan.step(j + k);
        if (pa.blend) pa.step[k].blend_t = (pa.step[k].a_kick - c->a[kA]) / (c->a[kB] - c->a[kA]);
      }
      rc = run_launch(c, pa, members);
      if (rc) return rc;
    }
    j0 = j1;
  }
  c->step_index = c->step_index + n;
  c->stepped = true;
  return FDF_OK;
}

// The workspace is carved deterministically, so fields and species added in
// the same order with the same sizes sit at the same device addresses: a graph
// captured for one such layout replays correctly after fdf_reset + re-adding,
// with other seeds too (a step reads them from the segment table).
std::vector<double> layout_signature(fdf_ctx* c) {
  std::vector<double> v;
  v.push_back((double)c->fields.size());
  for (auto& s : c->species) {
    v.push_back(s.field);
    v.push_back(s.m);
    v.push_back((double)s.n);
    v.push_back((double)s.flags);
  }
  return v;
}

HostStepState host_state(fdf_ctx* c) {
  HostStepState h;
  h.step_index = c->step_index;
  for (auto& s : c->species) {
    h.ints.insert(h.ints.end(), {s.cur, s.sorted ? 1 : 0, s.placed ? 1 : 0, s.order_time, s.pristine ? 1 : 0,
                                s.waited});
    h.drift_cells.push_back(s.drift_cells);
  }
  for (auto& f : c->fields) {
    h.grid_a.push_back(f.has_grid ? f.grid_a : NAN);
    h.ints.push_back(f.tag[0]);
    h.ints.push_back(f.tag[1]);
  }
  return h;
}

void apply_state(fdf_ctx* c, const HostStepState& h) {
  c->step_index = h.step_index;
  const int* v = h.ints.data();
  for (size_t i = 0; i < c->species.size(); ++i, v += 6) {
    c->species[i].cur = v[0];
    c->species[i].sorted = v[1] != 0;
    c->species[i].placed = v[2] != 0;
    c->species[i].order_time = v[3];
    c->species[i].pristine = v[4] != 0;
    c->species[i].waited = v[5];
    c->species[i].drift_cells = h.drift_cells[i];
  }
  for (size_t i = 0; i < c->fields.size(); ++i, v += 2) {
    c->fields[i].has_grid = !std::isnan(h.grid_a[i]);
    c->fields[i].grid_a = h.grid_a[i];
    c->fields[i].tag[0] = v[0];
    c->fields[i].tag[1] = v[1];
  }
  c->stepped = true;
}

// Graph mode: the launches of step(n) from a given host state are captured
// once (on a private stream) and replayed on the context stream afterwards.
int step_graph(fdf_ctx* c, int32_t n) {
  const HostStepState before = host_state(c);
  const std::vector<double> layout = layout_signature(c);
  for (auto& g : c->graphs) {
    if (g.n == n && g.before == before && g.layout == layout) {
      int rc = hip_check(c, hipGraphLaunch(g.exec, c->stream), "graph launch");
      if (!rc) apply_state(c, g.after);
      if (!rc && g.builds_grids) c->have_density = false;
      return rc;
    }
  }
  if (!c->cap_stream) {
    int rc = hip_check(c, hipStreamCreateWithFlags(&c->cap_stream, hipStreamNonBlocking), "capture stream");
    if (rc) return rc;
  }
  if (c->graphs.size() >= 16) clear_graphs(c);   // bounded cache
  GraphRec g;
  g.n = n;
  g.before = before;
  g.layout = layout;
  int rc = hip_check(c, hipStreamBeginCapture(c->cap_stream, hipStreamCaptureModeThreadLocal), "begin capture");
  if (rc) return rc;
  c->launch_stream = c->cap_stream;
  const bool density = c->have_density;
  c->have_density = true;   // a grid build clears it
  const int rc_enq = enqueue_steps(c, n);
  g.builds_grids = !c->have_density;
  c->have_density = density && !g.builds_grids;
  c->launch_stream = nullptr;
  rc = hip_check(c, hipStreamEndCapture(c->cap_stream, &g.graph), "end capture");
  if (rc_enq || rc) {
    if (g.graph) (void)hipGraphDestroy(g.graph);
    apply_state(c, before);
    return rc_enq ? rc_enq : rc;
  }
  rc = hip_check(c, hipGraphInstantiate(&g.exec, g.graph, nullptr, nullptr, 0), "graph instantiate");
  if (rc) {
    (void)hipGraphDestroy(g.graph);
    apply_state(c, before);
    return rc;
  }
  g.after = host_state(c);
  rc = hip_check(c, hipGraphLaunch(g.exec, c->stream), "graph launch");
  c->graphs.push_back(g);
  return rc;
}

}  // namespace

extern "C" {

int fdf_step(fdf_ctx* c, int32_t n) {
  if (!c) return FDF_ERR_ARG;
  if (!needs_ws(c)) return fail(c, FDF_ERR_WORKSPACE, "no workspace attached");
  if (c->species.empty()) return fail(c, FDF_ERR_STATE, "no species");
  if (n == 0) return FDF_OK;
  const int k0 = c->step_index;
  if (k0 + n < 0 || k0 + n > c->cfg.n_steps) return fail(c, FDF_ERR_ARG, "step range outside the schedule");
  int rc = upload_segments(c);
  if (rc) return rc;
  if (c->use_graph) return step_graph(c, n);
  return enqueue_steps(c, n);
}

int fdf_force_terms(fdf_ctx* c, int32_t sid, double* h_rms) {
  if (!c || !h_rms) return FDF_ERR_ARG;
  if (!needs_ws(c)) return fail(c, FDF_ERR_WORKSPACE, "no workspace attached");
  if (sid < 0 || sid >= (int)c->species.size()) return fail(c, FDF_ERR_ARG, "bad species id");
  const int s_gpsi = grid_slot(c->cfg, 0), s_gphi = grid_slot(c->cfg, 3), s_dot = grid_slot(c->cfg, 6);
  if (s_gpsi < 0 || s_gphi < 0 || s_dot == -2)
    return fail(c, FDF_ERR_UNSUPPORTED, "grad psi, grad phi and phi-dot are not all stored for this equation of motion");
  SpeciesRec& sp = c->species[sid];
  FieldRec& f = c->fields[sp.field];
  const double a = c->a[c->step_index];
  const bool tdep = c->cfg.potential_model == FDF_MODEL_RADMAT;
  if (!f.has_grid || (tdep && f.grid_a != a) || !c->anchors.empty()) {
    f.tag[0] = -1;   // buffer 0 no longer holds a super-step anchor
    const int rc = build_grid(c, sp.field, a);
    if (rc) return rc;
  }
  TermArgs t{};
  t.seg = sp.seg[sp.cur];
  t.fp64 = c->cfg.precision == FDF_PREC_FP64;
  t.G = c->cfg.grid_n;
  t.nslot = c->lay.nslot;
  t.slot_gpsi = s_gpsi;
  t.slot_gphi = s_gphi;
  t.slot_phidot = s_dot;
  t.box = c->cfg.box_mpc;
  t.ma = sp.m * a;
  t.grid = f.grid;
  t.out = (double*)(c->ws + c->lay.bins);
  launch_fill_zero(t.out, align_up(3 * kMaxBins * sizeof(double)), c->stream);
  std::pair<hipEvent_t, hipEvent_t> ev;
  timing_begin(c, FDF_KERNEL_OUTPUT, &ev);
  launch_force_terms(t, c->stream);
  timing_end(c, FDF_KERNEL_OUTPUT, ev);
  int rc = launched(c, "force terms");
  double sums[4];
  if (!rc) rc = hip_check(c, hipMemcpyAsync(sums, t.out, sizeof(sums), hipMemcpyDeviceToHost, c->stream), "terms");
  if (!rc) rc = hip_check(c, hipStreamSynchronize(c->stream), "terms");
  if (rc) return rc;
  for (int k = 0; k < 4; ++k) h_rms[k] = sp.n ? std::sqrt(sums[k] / (double)sp.n) : 0.0;
  return FDF_OK;
}

int fdf_weights(fdf_ctx* c, int32_t sid, double* d_w) {
  if (!c || !d_w) return FDF_ERR_ARG;
  if (sid < 0 || sid >= (int)c->species.size()) return fail(c, FDF_ERR_ARG, "bad species id");
  OutputArgs o = output_args(c, c->species[sid]);
  o.w_out = d_w;
  std::pair<hipEvent_t, hipEvent_t> ev;
  timing_begin(c, FDF_KERNEL_OUTPUT, &ev);
  launch_weights(o, c->stream);
  timing_end(c, FDF_KERNEL_OUTPUT, ev);
  return launched(c, "weights");
}

// Device buffers of one spectrum: the deposit halves (8 bytes per cell),
// the fixed-point deposit's largest |value|, the FFT planes (halves and the
// momentum spectrum's two accumulators), the FP32 form's binary32 halves and
// the bin accumulators.
struct PkBuffers {
  char* dens;
  uint32_t* max_bits;
  void* scratch;
  float* real32;
  double* bins;
};

// Arguments shared by both spectrum entry points; *G receives the mesh.
static int pk_validate(fdf_ctx* c, const int32_t* sp, int32_t ns, int32_t nbins, int32_t mode,
                       int32_t analysis_n, int* G) {
  if (!needs_ws(c)) return fail(c, FDF_ERR_WORKSPACE, "no workspace attached");
  if (nbins < 1 || nbins > kMaxBins) return fail(c, FDF_ERR_ARG, "n_bins must be in [1, 256]");
  if (mode != FDF_PK_CROSS && mode != FDF_PK_AUTO) return fail(c, FDF_ERR_ARG, "unknown mode");
  for (int i = 0; i < ns; ++i) {
    if (sp[i] < 0 || sp[i] >= (int)c->species.size()) return fail(c, FDF_ERR_ARG, "bad species id");
    // a total contrast only means something for species that see one field
    if (c->species[sp[i]].field != c->species[sp[0]].field)
      return fail(c, FDF_ERR_ARG, "the species of one spectrum must share a field");
    for (int j = 0; j < i; ++j)
      if (sp[j] == sp[i]) return fail(c, FDF_ERR_ARG, "a species is listed twice");
  }
  const int Gm = c->cfg.grid_n;
  if (analysis_n != 0 && (!is_pow2(analysis_n) || analysis_n < 8 || analysis_n > Gm))
    return fail(c, FDF_ERR_ARG, "analysis_n must be 0 or a power of two in [8, grid_n]");
  *G = analysis_n ? analysis_n : Gm;
  return FDF_OK;
}

// Binned spectrum of the energy-density contrast, or (momentum) of
// Theta = sum_a i k_a J_a with J the deposit of w q: the three axes are
// deposited and transformed one after the other and summed in Fourier space.
// Enqueues the work on the context stream; the bins end in b.bins as
// [count][sum |k|][sum P] per bin, from exact (order-independent) sums, and in
// means (if not null) as [mean |k|][mean P][count].  A small mesh's spectrum is
// bound by its launches: one fill for the three buffers, and the last block of
// the binning instead of launches after it (32^3, 32 K particles, FP32: 55 us
// with 14 launches, 41 us with 10).
static void pk_enqueue(fdf_ctx* c, const int32_t* sp, int32_t ns, int32_t nbins, int32_t mode,
                       bool momentum, int G, const PkBuffers& b, double* means) {
  const int Gm = c->cfg.grid_n;
  const bool f64 = c->cfg.precision == FDF_PREC_FP64;
  const size_t cells = (size_t)G * G * G;
  const double a = c->a[c->step_index];
  double esum = 0;
  for (int i = 0; i < ns; ++i) esum += mean_energy(c->species[sp[i]].m, a);
  // FP32 form: fixed-point halves in dens (int64 per cell), converted to
  // binary32 meshes for the transform
  int64_t n_all = 0;
  for (int i = 0; i < ns; ++i) n_all += c->species[sp[i]].n;
  int fixed_bits = 62;
  while (fixed_bits > 20 && ((int64_t)1 << (62 - fixed_bits)) < n_all) --fixed_bits;
  PkArgs pk{};
  pk.G = G;
  pk.fp64 = f64;
  pk.nbins = nbins;
  pk.auto_mode = mode == FDF_PK_AUTO;
  pk.volume = c->cfg.box_mpc * c->cfg.box_mpc * c->cfg.box_mpc;
  pk.grid_a = f64 ? (void*)b.dens : (void*)b.real32;
  pk.grid_b = f64 ? (void*)(b.dens + cells * 8) : (void*)(b.real32 + cells);
  pk.scratch = b.scratch;
  pk.twiddle = c->ws + (f64 ? c->lay.twiddle_d + twiddle_entry(Gm, G) * 16
                            : c->lay.twiddle_f + twiddle_entry(Gm, G) * 8);
  pk.bins = b.bins;
  pk.acc = (unsigned long long*)(b.bins + 3 * kMaxBins);
  pk.max_bits = (uint32_t*)(b.bins + 8 * kMaxBins);
  pk.ticket = pk.max_bits + 1;
  pk.means = means;
  pk.bin_plane = momentum ? 2 : 0;
  pk.kf = 2.0 * kPi / c->cfg.box_mpc;
  pk.deriv_axis = -1;
  for (int axis = momentum ? 0 : -1; axis < (momentum ? 3 : 0); ++axis) {
    const bool first = axis == (momentum ? 0 : -1);
    const FillArgs fill{{b.dens, b.max_bits, b.bins},
                        {align_up(2 * cells * 8), f64 ? 0 : kAlign, first ? align_up(kBinsBytes) : 0}};
    launch_fill_zero(fill, c->stream);
    for (int pass = f64 ? 1 : 0; pass < 2; ++pass)
    for (int i = 0; i < ns; ++i) {
      const SpeciesRec& s = c->species[sp[i]];
      OutputArgs o = output_args(c, s);
      o.auto_mode = mode == FDF_PK_AUTO;
      const double g3 = (double)cells;
      if (o.auto_mode) {
        o.norm[0] = o.norm[1] = g3 / ((double)s.n * esum);
      } else {
        const int64_t ne = (s.n + 1) / 2, no = s.n / 2;
        o.norm[0] = g3 / ((double)ne * esum);
        o.norm[1] = no ? g3 / ((double)no * esum) : 0.0;
      }
      o.G = G;
      o.dens[0] = b.dens;
      o.dens[1] = b.dens + cells * 8;
      o.quantity = axis;
      o.max_bits = b.max_bits;
      o.fixed_bits = fixed_bits;
      if (pass == 0) launch_deposit_max(o, c->stream);
      else launch_deposit(o, c->stream);
    }
    if (!f64) {
      FixedToRealArgs fr{};
      fr.src[0] = (const long long*)b.dens;
      fr.src[1] = (const long long*)(b.dens + cells * 8);
      fr.dst[0] = b.real32;
      fr.dst[1] = b.real32 + cells;
      fr.n_half = cells;
      fr.G = G;
      fr.n = (mode == FDF_PK_AUTO ? 1 : 2) * cells;
      fr.max_bits = b.max_bits;
      fr.fixed_bits = fixed_bits;
      launch_fixed_to_real(fr, c->stream);
    }
    pk.deriv_axis = axis;
    pk.accum_first = axis == 0;
    launch_power_spectrum(pk, c->stream);
  }
  launch_bin(pk, c->stream);
}

static int power_spectrum(fdf_ctx* c, const int32_t* sp, int32_t ns, int32_t nbins, int32_t mode,
                          bool momentum, int32_t analysis_n, double* hk, double* hp, double* hn) {
  if (!c || !sp || ns < 1 || !hk || !hp || !hn) return FDF_ERR_ARG;
  int G = 0;
  int rc = pk_validate(c, sp, ns, nbins, mode, analysis_n, &G);
  if (rc) return rc;
  PkBuffers b{};
  b.dens = c->ws + c->lay.dens;
  b.max_bits = (uint32_t*)(c->ws + c->lay.dep);
  b.scratch = c->ws + c->lay.scratch;
  b.real32 = (float*)(c->ws + c->lay.scratch + density_copy_offset(c));
  b.bins = (double*)(c->ws + c->lay.bins);
  std::pair<hipEvent_t, hipEvent_t> ev;
  timing_begin(c, FDF_KERNEL_OUTPUT, &ev);
  pk_enqueue(c, sp, ns, nbins, mode, momentum, G, b, nullptr);
  timing_end(c, FDF_KERNEL_OUTPUT, ev);
  rc = launched(c, "power spectrum");
  if (rc) return rc;
  double* const hb = c->pinned;
  rc = hip_check(c, hipMemcpyAsync(hb, b.bins, 3 * nbins * sizeof(double), hipMemcpyDeviceToHost, c->stream), "bins");
  if (!rc) rc = hip_check(c, hipStreamSynchronize(c->stream), "bins");
  if (rc) return rc;
  for (int i = 0; i < nbins; ++i) {
    const double cnt = hb[i];
    hn[i] = cnt;
    hk[i] = cnt > 0 ? hb[nbins + i] / cnt : NAN;
    hp[i] = cnt > 0 ? hb[2 * nbins + i] / cnt : NAN;
  }
  c->have_density = !momentum && G == c->cfg.grid_n;   // else the buffers hold another quantity or mesh
  c->density_auto = mode == FDF_PK_AUTO;
  return FDF_OK;
}

int fdf_density_power_spectrum(fdf_ctx* c, const int32_t* sp, int32_t ns, int32_t nbins, int32_t mode,
                               double* hk, double* hp, double* hn) {
  return power_spectrum(c, sp, ns, nbins, mode, false, 0, hk, hp, hn);
}

int fdf_momentum_power_spectrum(fdf_ctx* c, const int32_t* sp, int32_t ns, int32_t nbins, int32_t mode,
                                double* hk, double* hp, double* hn) {
  return power_spectrum(c, sp, ns, nbins, mode, true, 0, hk, hp, hn);
}

int fdf_power_spectrum(fdf_ctx* c, const int32_t* sp, int32_t ns, int32_t nbins, int32_t mode,
                       int32_t quantity, int32_t analysis_n, double* hk, double* hp, double* hn) {
  if (quantity != FDF_PK_DENSITY && quantity != FDF_PK_MOMENTUM)
    return c ? fail(c, FDF_ERR_ARG, "unknown quantity") : FDF_ERR_ARG;
  return power_spectrum(c, sp, ns, nbins, mode, quantity == FDF_PK_MOMENTUM, analysis_n, hk, hp, hn);
}

int fdf_power_spectrum_noalloc(fdf_ctx* c, const int32_t* sp, int32_t ns, int32_t nbins, int32_t mode,
                               int32_t quantity, int32_t analysis_n, double* d_out) {
  if (!c || !sp || ns < 1 || !d_out) return FDF_ERR_ARG;
  if (quantity != FDF_PK_DENSITY && quantity != FDF_PK_MOMENTUM) return fail(c, FDF_ERR_ARG, "unknown quantity");
  int G = 0;
  int rc = pk_validate(c, sp, ns, nbins, mode, analysis_n, &G);
  if (rc) return rc;
  const bool f64 = c->cfg.precision == FDF_PREC_FP64;
  if (G > kStaticMaxMesh || static_scratch_bytes(f64, G) > kStaticScratchBytes)
    return fail(c, FDF_ERR_ARG, "the no-allocation spectrum needs an analysis mesh of at most 64^3 "
                                "(analysis_n in [8, 64]): its static scratch holds 16 MiB");
  char* st = nullptr;
  rc = static_scratch(c, &st);
  if (rc) return rc;
  const size_t g3 = (size_t)G * G * G, plane = (size_t)G * G * (G / 2) * (f64 ? 16 : 8);
  PkBuffers b{};
  size_t off = 0;
  b.bins = (double*)(st + off); off += align_up(kBinsBytes);
  b.max_bits = (uint32_t*)(st + off); off += kAlign;
  b.dens = st + off; off += align_up(2 * g3 * 8);
  b.scratch = st + off; off += align_up(4 * plane);
  b.real32 = f64 ? nullptr : (float*)(st + off);
  pk_enqueue(c, sp, ns, nbins, mode, quantity == FDF_PK_MOMENTUM, G, b, d_out);
  return launched(c, "power spectrum (static scratch)");
}

// State of a species that is in the order of its ids, array by array.
static int read_state_arrays(fdf_ctx* c, const SpeciesRec& s, double* hx, double* hq) {
  const Segment& g = s.seg[s.cur];
  const bool f64 = c->cfg.precision == FDF_PREC_FP64;
  const int64_t piece = std::min<int64_t>(s.n, 1 << 20);
  std::vector<double> d(f64 ? piece : 0);
  std::vector<float> q0(f64 ? 0 : piece), dq(f64 ? 0 : piece);
  std::vector<uint32_t> u(f64 ? 0 : piece);
  auto get = [&](auto& to, const auto* from, int64_t n) {
    return hip_check(c, hipMemcpy(to.data(), from, n * sizeof(*from), hipMemcpyDeviceToHost), "read state");
  };
  int rc = hip_check(c, hipStreamSynchronize(c->stream), "sync");
  for (int64_t i0 = 0; i0 < s.n; i0 += piece) {
    const int64_t n = std::min(piece, s.n - i0);
    for (int k = 0; k < 3; ++k) {
      if (hx && !rc) {
        double* const h = hx + 3 * i0 + k;
        rc = f64 ? get(d, g.xd[k] + i0, n) : get(u, g.xu[k] + i0, n);
        for (int64_t i = 0; i < n; ++i) h[3 * i] = f64 ? d[i] : (double)u[i] * (c->cfg.box_mpc * 0x1p-32);
      }
      if (hq && !rc) {
        double* const h = hq + 3 * i0 + k;
        rc = f64 ? get(d, g.qd[k] + i0, n) : get(q0, g.q0f[k] + i0, n);
        if (!f64 && !rc) rc = get(dq, g.dqf[k] + i0, n);
        for (int64_t i = 0; i < n; ++i) h[3 * i] = f64 ? d[i] : (double)q0[i] + (double)dq[i];
      }
      if (rc) return rc;
    }
  }
  return rc;
}

// Ids of a slice below which fdf_read_state copies the arrays instead of reading
// several slices (a slice costs a launch, a copy and a scan of all ids for the
// positions and again for the momenta).  1 M particles, slices against arrays:
// 341 ids (8^3, FP32) 96 and 6.1 ms, 2730 (16^3, FP32) 21 and 6.1, 9557 (16^3,
// FP64) 7.6 and 6.4, 21845 (32^3, FP32) 4.6 and 6.1, 76458 (32^3, FP64) 3.2 and
// 6.4; 10 K particles in 341 1.03 and 0.25.
constexpr int64_t kReadSliceIds = 16384;

int fdf_read_state(fdf_ctx* c, int32_t sid, double* hx, double* hq) {
  if (!c) return FDF_ERR_ARG;
  if (sid < 0 || sid >= (int)c->species.size()) return fail(c, FDF_ERR_ARG, "bad species id");
  const SpeciesRec& s = c->species[sid];
  // A kernel puts the state in id order: in the species' other copy, which holds
  // nothing between the steps, or without one in the FFT scratch (FP32: below
  // the density copy), in slices of ids that fit.  The scratch grows with the
  // mesh alone, so a small one takes many slices; a species there is in id
  // order (nothing re-orders it on a mesh that the L2 holds) and its arrays can
  // be copied instead.
  ReadStateArgs a{};
  a.seg = s.seg[s.cur];
  a.fp64 = c->cfg.precision == FDF_PREC_FP64;
  a.box = c->cfg.box_mpc;
  a.out = (double*)(c->ws + c->lay.scratch);
  size_t room = a.fp64 ? c->lay.scratch_bytes : density_copy_offset(c);
  if (c->cfg.sort_every > 0) {
    const Segment& o = s.seg[s.cur ^ 1];   // its arrays, from the first to the ids, in one piece
    char* const first = a.fp64 ? (char*)o.xd[0] : (char*)o.xu[0];
    a.out = (double*)first;
    room = (size_t)((char*)(o.id + s.n) - first);
  }
  const int64_t slice = (int64_t)(room / (3 * sizeof(double)));
  if (s.n > slice && slice < kReadSliceIds && !s.sorted) return read_state_arrays(c, s, hx, hq);
  for (int m = 0; m < 2; ++m) {
    double* h = m ? hq : hx;
    if (!h) continue;
    a.momenta = m;
    for (a.first = 0; a.first < s.n; a.first += slice) {
      a.count = std::min<int64_t>(slice, s.n - a.first);
      launch_read_state(a, c->stream);
      int rc = launched(c, "read state");
      if (!rc)
        rc = hip_check(c, hipMemcpyAsync(h + 3 * a.first, a.out, (size_t)a.count * 3 * sizeof(double),
                                         hipMemcpyDeviceToHost, c->stream), "read state");
      if (rc) return rc;
    }
  }
  return hip_check(c, hipStreamSynchronize(c->stream), "sync");
}

int fdf_read_grid(fdf_ctx* c, int32_t field_id, int32_t slot, double* h) {
  if (!c || !h) return FDF_ERR_ARG;
  if (field_id < 0 || field_id >= (int)c->fields.size()) return fail(c, FDF_ERR_ARG, "bad field id");
  if (slot < 0 || slot > 9) return fail(c, FDF_ERR_ARG, "quantity must be in [0, 9]");
  const FieldRec& f = c->fields[field_id];
  if (!f.has_grid) return fail(c, FDF_ERR_STATE, "grid not built");
  const int ns = c->lay.nslot;
  const int s = grid_slot(c->cfg, slot);
  if (s == -2) return fail(c, FDF_ERR_UNSUPPORTED, "quantity not stored for this equation of motion");
  if (s == -1) {
    std::fill(h, h + (size_t)c->cfg.grid_n * c->cfg.grid_n * c->cfg.grid_n, 0.0);
    return FDF_OK;
  }
  const size_t cells = (size_t)c->cfg.grid_n * c->cfg.grid_n * c->cfg.grid_n;
  const bool f64 = c->cfg.precision == FDF_PREC_FP64;
  int rc = hip_check(c, hipStreamSynchronize(c->stream), "sync");
  if (rc) return rc;
  // the device mesh is bricked (mesh_x/y/z); the host array is x-major
  const uint32_t G = (uint32_t)c->cfg.grid_n;
  std::vector<size_t> where(cells);
  for (uint32_t ix = 0; ix < G; ++ix)
    for (uint32_t iy = 0; iy < G; ++iy)
      for (uint32_t iz = 0; iz < G; ++iz)
        where[((size_t)ix * G + iy) * G + iz] = (size_t)mesh_x(ix, G) + mesh_y(iy, G) + mesh_z(iz);
  if (f64) {
    std::vector<double> all(cells * ns);
    rc = hip_check(c, hipMemcpy(all.data(), f.grid, all.size() * 8, hipMemcpyDeviceToHost), "read grid");
    for (size_t i = 0; i < cells && !rc; ++i) h[i] = all[where[i] * ns + s];
  } else {
    std::vector<uint16_t> all(cells * ns);
    rc = hip_check(c, hipMemcpy(all.data(), f.grid, all.size() * 2, hipMemcpyDeviceToHost), "read grid");
    for (size_t i = 0; i < cells && !rc; ++i) {
      uint32_t u = (uint32_t)all[where[i] * ns + s] << 16;
      float v;
      std::memcpy(&v, &u, 4);
      h[i] = v;
    }
  }
  return rc;
}

int fdf_read_field(fdf_ctx* c, int32_t field_id, double* h) {
  if (!c || !h) return FDF_ERR_ARG;
  if (field_id < 0 || field_id >= (int)c->fields.size()) return fail(c, FDF_ERR_ARG, "bad field id");
  const int G = c->cfg.grid_n, M = G / 2, H = M + 1;
  const bool f64 = c->cfg.precision == FDF_PREC_FP64;
  const size_t n = (size_t)G * G * M * 2;
  std::vector<double> d(n);
  std::vector<float> f(f64 ? 0 : n);
  int rc = hip_check(c, hipStreamSynchronize(c->stream), "sync");
  if (!rc) rc = hip_check(c, hipMemcpy(f64 ? (void*)d.data() : (void*)f.data(), c->fields[field_id].dk,
                                       n * (f64 ? 8 : 4), hipMemcpyDeviceToHost), "read field");
  if (rc) return rc;
  if (!f64) for (size_t i = 0; i < n; ++i) d[i] = f[i];
  for (int ix = 0; ix < G; ++ix)
    for (int iy = 0; iy < G; ++iy)
      for (int iz = 0; iz < H; ++iz) {
        const size_t dst = (((size_t)ix * G + iy) * H + iz) * 2;
        if (iz == M) { h[dst] = 0; h[dst + 1] = 0; continue; }
        const size_t src = (((size_t)ix * G + iy) * M + iz) * 2;
        h[dst] = d[src];
        h[dst + 1] = d[src + 1];
      }
  return FDF_OK;
}

int fdf_read_density(fdf_ctx* c, int32_t half, double* h) {
  if (!c || !h) return FDF_ERR_ARG;
  if (!c->have_density) return fail(c, FDF_ERR_STATE, "no density deposited yet");
  if (half < 0 || half > 1) return fail(c, FDF_ERR_ARG, "half must be 0 or 1");
  const size_t cells = (size_t)c->cfg.grid_n * c->cfg.grid_n * c->cfg.grid_n;
  const bool f64 = c->cfg.precision == FDF_PREC_FP64;
  const char* src = f64 ? c->ws + c->lay.dens + half * cells * 8
                        : c->ws + c->lay.scratch + density_copy_offset(c) + half * cells * 4;
  int rc = hip_check(c, hipStreamSynchronize(c->stream), "sync");
  if (rc) return rc;
  if (f64) return hip_check(c, hipMemcpy(h, src, cells * 8, hipMemcpyDeviceToHost), "read density");
  std::vector<float> f(cells);
  rc = hip_check(c, hipMemcpy(f.data(), src, cells * 4, hipMemcpyDeviceToHost), "read density");
  for (size_t i = 0; i < cells && !rc; ++i) h[i] = f[i];
  return rc;
}

int fdf_read_schedule(const fdf_ctx* c, double* h) {
  if (!c || !h) return FDF_ERR_ARG;
  const int n = c->cfg.n_steps;
  std::copy(c->a.begin(), c->a.end(), h);
  std::copy(c->a_half.begin(), c->a_half.end(), h + n + 1);
  std::copy(c->kick1.begin(), c->kick1.end(), h + 2 * n + 1);
  std::copy(c->kick2.begin(), c->kick2.end(), h + 3 * n + 1);
  std::copy(c->drift.begin(), c->drift.end(), h + 4 * n + 1);
  return FDF_OK;
}

int fdf_get_info(const fdf_ctx* c, fdf_info* info) {
  if (!c || !info) return FDF_ERR_ARG;
  std::memset(info, 0, sizeof(*info));
  info->step_index = c->step_index;
  info->n_steps = c->cfg.n_steps;
  info->a_current = c->a[c->step_index];
  info->amplitude = c->amp;
  info->tau_begin = c->tau_begin;
  info->n_fields = (int32_t)c->fields.size();
  info->n_species = (int32_t)c->species.size();
  for (auto& s : c->species) info->n_particles += s.n;
  info->workspace_used = c->lay.total;
  return FDF_OK;
}

int fdf_get_tuning(const fdf_ctx* c, fdf_tuning* t) {
  if (!c || !t) return FDF_ERR_ARG;
  std::memset(t, 0, sizeof(*t));
  t->particles_per_thread = c->ppt;
  t->sort_tiles = c->sort_tiles;
  t->sort_every = c->sort_every;
  t->sort_cells = c->sort_cells;
  t->persistent_blocks = c->persistent;
  t->use_graph = c->use_graph ? 1 : 0;
  t->sort_predict = c->sort_predict ? 1 : 0;
  t->sort_fused = c->sort_fused ? 1 : 0;
  t->push_waves = c->push_waves;
  t->sort_push_ppt = c->sort_push_ppt;
  t->sort_keys_push = c->sort_keys_push ? 1 : 0;
  return FDF_OK;
}

int fdf_set_tuning(fdf_ctx* c, const fdf_tuning* t) {
  if (!c || !t) return FDF_ERR_ARG;
  const int p = t->particles_per_thread;
  if (p != 1 && p != 2 && p != 4 && p != 8) return fail(c, FDF_ERR_ARG, "particles_per_thread must be 1, 2, 4 or 8");
  const int tmax = std::min(c->cfg.grid_n, 256);
  if (t->sort_tiles != 0 && (!is_pow2(t->sort_tiles) || t->sort_tiles > tmax))
    return fail(c, FDF_ERR_ARG, "sort_tiles must be 0 or a power of two <= min(G, 256)");
  if (t->sort_every < 0 || (t->sort_every > 0 && c->cfg.sort_every == 0))
    return fail(c, FDF_ERR_ARG, "sorting needs a context created with sort_every > 0");
  if (!(t->sort_cells >= 0) || (t->sort_cells > 0 && c->cfg.sort_every == 0))
    return fail(c, FDF_ERR_ARG, "sort_cells must be >= 0 (and > 0 needs sort_every > 0 at create)");
  if (t->persistent_blocks < 0 || t->persistent_blocks % 8 != 0 || t->persistent_blocks > (1 << 20))
    return fail(c, FDF_ERR_ARG, "persistent_blocks must be 0 or a positive multiple of 8");
  if (t->use_graph != 0 && t->use_graph != 1) return fail(c, FDF_ERR_ARG, "use_graph must be 0 or 1");
  if (t->sort_predict != 0 && t->sort_predict != 1) return fail(c, FDF_ERR_ARG, "sort_predict must be 0 or 1");
  if (t->sort_fused != 0 && t->sort_fused != 1) return fail(c, FDF_ERR_ARG, "sort_fused must be 0 or 1");
  if (t->push_waves != 0 && (t->push_waves < 2 || t->push_waves > 8))
    return fail(c, FDF_ERR_ARG, "push_waves must be 0 or in [2, 8]");
  if (t->sort_push_ppt != 0 && t->sort_push_ppt != 1 && t->sort_push_ppt != 2 && t->sort_push_ppt != 4)
    return fail(c, FDF_ERR_ARG, "sort_push_ppt must be 0, 1, 2 or 4");
  if (t->sort_keys_push != 0 && t->sort_keys_push != 1) return fail(c, FDF_ERR_ARG, "sort_keys_push must be 0 or 1");
  clear_graphs(c);
  c->persistent = t->persistent_blocks;
  c->use_graph = t->use_graph != 0;
  c->ppt = p;
  c->sort_tiles = t->sort_tiles;
  c->sort_every = t->sort_every;
  c->sort_cells = t->sort_cells;
  c->sort_predict = t->sort_predict != 0;
  c->sort_fused = t->sort_fused != 0;
  c->push_waves = t->push_waves;
  c->sort_push_ppt = t->sort_push_ppt ? t->sort_push_ppt : 4;
  c->sort_keys_push = t->sort_keys_push != 0;
  return FDF_OK;
}

int fdf_sync(fdf_ctx* c) {
  if (!c) return FDF_ERR_ARG;
  return hip_check(c, hipStreamSynchronize(c->stream), "sync");
}

int fdf_timing_enable(fdf_ctx* c, int32_t on) {
  if (!c) return FDF_ERR_ARG;
  c->timing = on != 0;
  return FDF_OK;
}

int fdf_read_timing(fdf_ctx* c, int32_t cls, double* ms, int64_t* launches) {
  if (!c || !ms || !launches) return FDF_ERR_ARG;
  if (cls < 0 || cls >= FDF_KERNEL_COUNT) return fail(c, FDF_ERR_ARG, "bad kernel class");
  timing_collect(c);
  *ms = c->tim[cls].total_ms;
  *launches = c->tim[cls].launches;
  return FDF_OK;
}

int fdf_timing_reset(fdf_ctx* c) {
  if (!c) return FDF_ERR_ARG;
  timing_collect(c);
  for (auto& t : c->tim) { t.total_ms = 0; t.launches = 0; t.work[0] = t.work[1] = t.work[2] = t.passes[0] = t.passes[1] = 0; }
  return FDF_OK;
}

int fdf_read_work(fdf_ctx* c, int32_t cls, int64_t* work) {
  if (!c || !work) return FDF_ERR_ARG;
  if (cls < 0 || cls >= FDF_KERNEL_COUNT) return fail(c, FDF_ERR_ARG, "bad kernel class");
  for (int k = 0; k < 3; ++k) work[k] = c->tim[cls].work[k];
  return FDF_OK;
}

int fdf_read_passes(fdf_ctx* c, int32_t cls, int64_t* passes) {
  if (!c || !passes) return FDF_ERR_ARG;
  if (cls < 0 || cls >= FDF_KERNEL_COUNT) return fail(c, FDF_ERR_ARG, "bad kernel class");
  for (int k = 0; k < 2; ++k) passes[k] = c->tim[cls].passes[k];
  return FDF_OK;
}

}  // extern "C"
