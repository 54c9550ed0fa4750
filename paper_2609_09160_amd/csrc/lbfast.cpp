// lbfast.cpp -- host runtime behind the C ABI of include/lbfast.h: argument
// validation, buffer ownership, flip/flop bookkeeping (the paper's two
// ten-field arrays, section 3), launch shape, conversions and reductions.
#include "lbfast.h"
#include "lbfast_measure.h"

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <algorithm>
#include <cstring>
#include <new>
#include <string>

#include "internal.hpp"

namespace lbf {
// measurement utilities, aux.hip
hipError_t launch_copy_probe(const void* src, void* dst, int64_t n4, hipStream_t s);
hipError_t launch_planes_probe(const void* src, void* dst, int64_t n, int nplanes, hipStream_t s);
hipError_t launch_zmarch_probe(const void* src, void* dst, int nx, int ny, int nz, int layout,
                               int zchunk, hipStream_t s);
}  // namespace lbf

namespace {

thread_local std::string g_err;

int fail(int code, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  g_err = buf;
  return code;
}

}  // namespace

// error reporting for entry points defined in other translation units
namespace lbf {
void clear_error() { g_err.clear(); }
int set_error(int code, const char* msg) {
  g_err = msg;
  return code;
}
}  // namespace lbf

namespace {

int hip_fail(hipError_t e, const char* what) {
  return fail(LBF_E_DEVICE, "%s: %s (%d)", what, hipGetErrorString(e), static_cast<int>(e));
}

size_t elem_bytes(int storage) {
  switch (storage) {
    case LBF_F64: return 8;
    case LBF_F32: return 4;
    case LBF_F16S:
    case LBF_BF16S:
    case LBF_F16SU: return 2;
    default: return 0;
  }
}

// planes of one state buffer: the ten moments, plus the three low velocity
// words of the split form
size_t state_planes(int storage) { return storage == LBF_F16SU ? 13 : 10; }

bool is_16bit(int storage) {
  return storage == LBF_F16S || storage == LBF_BF16S || storage == LBF_F16SU;
}

bool is_pow2_float(float s) {
  if (!(s > 0.0f) || !std::isfinite(s)) return false;
  int e;
  return std::frexp(s, &e) == 0.5f;
}

int validate(const lbfast_params* p) {
  if (!p) return fail(LBF_E_ARG, "params is NULL");
  if (p->struct_size != sizeof(lbfast_params))
    return fail(LBF_E_ARG, "params.struct_size = %u, expected %zu", p->struct_size,
                sizeof(lbfast_params));
  if (p->lattice != LBF_D3Q19 && p->lattice != LBF_D3Q27 && p->lattice != LBF_D3Q27H)
    return fail(LBF_E_ARG, "lattice must be LBF_D3Q19, LBF_D3Q27 or LBF_D3Q27H (got %d)",
                p->lattice);
  if (elem_bytes(p->storage) == 0) return fail(LBF_E_ARG, "unknown storage %d", p->storage);
  const int64_t n[3] = {p->nx, p->ny, p->nz};
  for (int a = 0; a < 3; ++a) {
    if (n[a] < 1) return fail(LBF_E_ARG, "grid extent %d is %lld (must be >= 1)", a,
                              static_cast<long long>(n[a]));
    if (n[a] > (1 << 30)) return fail(LBF_E_ARG, "grid extent %d too large", a);
    if (p->bc[a] != LBF_PERIODIC && p->bc[a] != LBF_WALLS)
      return fail(LBF_E_ARG, "bc[%d] = %d is not LBF_PERIODIC/LBF_WALLS", a, p->bc[a]);
  }
  if (p->bc[0] == LBF_WALLS || p->bc[2] == LBF_WALLS)
    return fail(LBF_E_UNSUPPORTED, "walls are supported on the y axis only");
  if (p->bc[1] == LBF_WALLS && p->ny < 2)
    return fail(LBF_E_ARG, "a walled axis needs at least 2 sites (ny = %lld)",
                static_cast<long long>(p->ny));
  const double N = static_cast<double>(p->nx) * static_cast<double>(p->ny) * static_cast<double>(p->nz);
  if (N > 4.0e9) return fail(LBF_E_ARG, "grid has %.3g sites (limit 4e9)", N);
  // in-plane byte offsets are 32-bit in the kernels (8-byte elements worst case)
  if (static_cast<double>(p->nx) * static_cast<double>(p->ny) * 8.0 >= 4294967296.0)
    return fail(LBF_E_ARG, "nx*ny too large (an x-y plane of 8-byte values must fit in 4 GiB)");
  if (!(p->tau > 0.5) || !std::isfinite(p->tau))
    return fail(LBF_E_ARG, "tau must be a finite value > 1/2 (got %g)", p->tau);
  for (int a = 0; a < 3; ++a)
    if (!std::isfinite(p->force[a])) return fail(LBF_E_ARG, "force[%d] is not finite", a);
  const bool s16 = is_16bit(p->storage);
  for (int k = 0; k < 10; ++k) {
    if (p->scale[k] == 0.0f) continue;
    if (!s16) return fail(LBF_E_ARG, "scale[] is only meaningful for 16-bit storage");
    if (!is_pow2_float(p->scale[k]))
      return fail(LBF_E_ARG, "scale[%d] = %g is not a positive power of two", k, p->scale[k]);
  }
  for (int k = 0; k < 7; ++k)
    if (p->reserved[k] != 0) return fail(LBF_E_ARG, "reserved[%d] must be zero", k);
  if (p->rounding != LBF_ROUND_AUTO && p->rounding != LBF_ROUND_NEAREST &&
      p->rounding != LBF_ROUND_STOCHASTIC)
    return fail(LBF_E_ARG, "rounding must be LBF_ROUND_AUTO, _NEAREST or _STOCHASTIC");
  if (p->rounding == LBF_ROUND_STOCHASTIC && !s16)
    return fail(LBF_E_ARG, "stochastic rounding applies to 16-bit storage only");
  if (p->storage == LBF_F16SU && p->rounding == LBF_ROUND_STOCHASTIC)
    return fail(LBF_E_ARG, "LBF_F16SU rounds to nearest (its velocity keeps 22 bits)");
  return LBF_OK;
}

}  // namespace

// Launch geometry of a step or an adjoint step
struct Launch {
  int slab, cached, xcd_remap;       // as in lbf::StepArgs
  int lane_sites, rows;
  int tiles_x, tiles_y, zchunk, zchunks;
};

struct lbfast_ctx {
  lbfast_params p;
  int device = 0;
  hipStream_t stream = nullptr;
  void* buf[2] = {nullptr, nullptr};
  bool owned = false;
  int cur = 0;
  const void* Ffield = nullptr;
  float scale[10];
  float inv_scale[10];
  bool scales_fixed = false;
  int tile_rows = 8;       // launch shape once the caller has chosen rows or sites
  int lane_sites = 1;
  bool shape_set = false;
  int auto_sites = 1, auto_rows = 4;  // launch shape until then
  bool auto_slab = false;             // one plane per workgroup instead (no z_chunk set)
  int z_chunk = 0;
  bool two_phase = false;
  lbfast_phase_params pp;
  void* phi[2] = {nullptr, nullptr};  // phase field, two time levels
  void* Fph[2] = {nullptr, nullptr};  // force of the two time levels (3 planes)
  int pcur = 0;
  double* d_partials = nullptr;  // kReduceBlocks*5 + 5 doubles
  unsigned* d_maxbits = nullptr; // 10
  int64_t N = 0;
  uint64_t steps_done = 0;       // steps since create: seeds the stochastic rounding
  int adj_sites = 0, adj_rows = 0;  // adjoint launch shape (0: automatic)
  int block_order = 0;              // 0 automatic, 1 hardware order, 2 per-XCD ranges
  int form = LBF_FORM_AUTO;         // march or one-plane form of the steps
  // What the settings above come to, kept so that a call of few steps does not
  // evaluate the launch model: see plan()
  Launch step;
  lbf::PassGeom phase, force;       // two-component variant
  int cus = 256;                    // compute units of the device
};

namespace {

int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// LDS of one step workgroup: staged populations x (rows + 2) x (64 S + 2)
// columns, plus the x-halo column buffer
// LDS of one step workgroup; the two-component step stages phi(t+1) in one
// more slot for its stencils
size_t lds_bytes(int Q, int storage, int tile_rows, int lane_sites, bool stencil = false) {
  const size_t np = ((Q == LBF_D3Q19) ? 16 : 24) + (stencil ? 1 : 0);
  const size_t c = (storage == LBF_F64) ? 8 : 4;
  return c * np * static_cast<size_t>(tile_rows + 2) * static_cast<size_t>(64 * lane_sites + 4);
}
constexpr size_t kLdsLimit = 160 * 1024;

// What decides the time of one march (a step or an adjoint step) besides its
// launch shape.
struct MarchForm {
  int Q, storage;
  bool stencil;          // one more LDS slot (two-component step)
  int cus;               // compute units of the device
  double read, write;    // bytes per site
  int streams;           // separate arrays read at an x-halo site
  bool cached_forms;     // there are kernels with plain stores (step_cached)
  double l0, l1, busy;   // us per plane, see march_us
  double slab, slab_mem; // one-plane form, see slab_us
};

// Both state buffers within the 256 MB last-level cache, with room for the
// rest: stores then leave the new state there (plain stores).  Measured where
// it turns: FP32 144^3 (2 x 119 MB) 84 us with plain stores against 87 with
// non-temporal ones, 160^3 (2 x 164 MB) 95 against 91.
constexpr double kCacheStateBytes = 120e6;

bool fits_cache(const lbfast_ctx* h) {
  return static_cast<double>(lbfast_buffer_bytes(&h->p)) <= kCacheStateBytes;
}

// phases of unequal density or viscosity, or a density other than 1: the
// step reads the phase field for a density and relaxation rate per site
bool variable_properties(const lbfast_ctx* h) {
  return h->pp.rho_l != 1.0 || h->pp.rho_h != 1.0 || h->pp.tau_l != h->pp.tau_h;
}

// 16-bit forms whose stored words depend on the launch: the compiler contracts
// FP32 differently in the two copies of a plane in the march's unrolled loop
// (even and odd planes of a chunk) and, for some, between tile heights.  One
// such difference moves a 16-bit word now and then, and BF16's stochastic
// rounding makes every one a step of 2^-8.  FP16 with D3Q19 and D3Q27 is free of
// both.  The others keep the parity of the planes that the chunks of
// width_zchunk give, and where more than that matters these chunks themselves
// and the rows of width_launch (BF16 D3Q19 48 x 104 x 46: 0.07% off after 29
// steps in chunks of another even length).  FP16SU with D3Q19 and D3Q27 keeps
// the parity alone, which its words need without a force; with a uniform force
// low words of the velocity differ between tile heights (27 of 100 drawn grids
// after 6 steps, at most 8e-4 of a state, 7e-8 of its largest value), which is
// accepted: held to the 8 rows of width_launch, it took up to 1.6 times as long
// (168 x 232 x 63 D3Q27 50.6 us, 82.0).
bool keeps_parity(const lbfast_ctx* h) {
  return is_16bit(h->p.storage) &&
         (h->p.storage != LBF_F16S || h->p.lattice == LBF_D3Q27H || h->two_phase);
}
bool keeps_rows(const lbfast_ctx* h) {
  return keeps_parity(h) &&
         !(h->p.storage == LBF_F16SU && h->p.lattice != LBF_D3Q27H && !h->Ffield);
}

// States of at least a few MB gain from what the cache keeps (plain stores,
// contiguous tile ranges per XCD); smaller ones lose a little (64^3 FP32, 10.5
// MB: 9.0 us non-temporal, 9.3 plain; 10.0 contiguous; FP16 32 x 136 x 224, 20
// MB, 1.6% slower with both, 112^3, 28 MB, 5% faster).
bool cache_matters(const lbfast_ctx* h) {
  const double least = is_16bit(h->p.storage) ? 24e6 : 11e6;
  return fits_cache(h) && static_cast<double>(lbfast_buffer_bytes(&h->p)) >= least;
}

// Whether a step in this shape stores plainly.  Not the 16-bit forms that keep
// their rows, but for BF16 with D3Q19 and D3Q27: there the kernels with plain
// stores are contracted differently, too.
bool step_cached(const lbfast_ctx* h, int S, int ty) {
  return cache_matters(h) && !h->two_phase && lbf::march_cached(S, ty) &&
         (!keeps_rows(h) || (h->p.storage == LBF_BF16S && h->p.lattice != LBF_D3Q27H));
}

MarchForm march_form(const lbfast_ctx* h, bool adjoint = false) {
  MarchForm f{};
  f.Q = h->p.lattice;
  f.storage = h->p.storage;
  f.stencil = h->two_phase;
  f.cus = h->cus;
  const double e = static_cast<double>(elem_bytes(f.storage));
  const double c = f.storage == LBF_F64 ? 8.0 : 4.0;
  f.read = f.write = static_cast<double>(state_planes(f.storage)) * e;
  f.streams = f.storage == LBF_F16SU ? 4 : (is_16bit(f.storage) ? 3 : 10);
  if (h->Ffield || h->two_phase) f.read += 3 * c, f.streams += 3;
  if (h->two_phase) f.read += c, f.write += 3 * c, f.streams += 1;
  if (adjoint) f.read = 22 * c, f.write = 13 * c, f.streams = 13, f.stencil = false;
  f.cached_forms = !adjoint;
  const bool c64 = c == 8.0, q19 = f.Q == LBF_D3Q19, full = f.Q == LBF_D3Q27H;
  f.slab = q19 ? (c64 ? 12.0 : 11.5) : full ? (c64 ? 15.0 : 13.5) : (c64 ? 12.0 : 10.0);
  if (f.stencil)
    f.slab += full ? 0.5 : c64 ? 3.0 : 2.5;
  else if (h->Ffield && q19)
    f.slab += c64 ? 2.0 : 1.0;
  f.slab_mem = c * ((f.stencil ? 70 : h->Ffield ? 50 : 30) + (full ? 20 : 0));
  if (adjoint) f.slab = c64 ? 12.0 : 10.0, f.slab_mem = 80 * c;
  // fitted to the times of 50 to 900 launch shapes per grid (9 x 16 x 17 to
  // 512^3), per velocity set and compute type
  const bool f64 = f.storage == LBF_F64;
  if (f.Q == LBF_D3Q19) {
    f.l0 = 0.45, f.l1 = f64 ? 0.15 : 0.07, f.busy = f64 ? 0.19 : 0.09;
  } else if (f.Q == LBF_D3Q27) {
    f.l0 = f64 ? 0.8 : 0.6, f.l1 = f64 ? 0.185 : 0.1, f.busy = f64 ? 0.3 : 0.135;
  } else {
    f.l0 = f64 ? 1.3 : 1.15, f.l1 = f64 ? 0.2 : 0.045, f.busy = f64 ? 0.37 : 0.175;
  }
  // the stencils of the two-component step, and the adjoint's 22 values per
  // site (see slab_us), by the same measure
  const double heavier = h->two_phase ? 1.25 : (adjoint ? 1.65 : 1.0);
  f.l0 *= heavier, f.l1 *= heavier, f.busy *= heavier;
  return f;
}

// Modelled time in us of a march with S sites per lane, ty tile rows and
// z-chunks of zc planes (up to a constant).  A workgroup runs zc + 2 planes (an
// even number); alone on a CU a plane takes l0 + l1 S (ty + 1) (latency and
// barriers), and n workgroups on one CU at least n busy S (ty + 1) (issue), so
// that what counts is the number of workgroups on the fullest of the 256 CUs:
// grids run best in one wave of at most 256.  Against that stands the memory:
// the planes and their y and z halos, 128 bytes for every x-halo site and
// stream, read at 9 TB/s, and the stores at 5.6 TB/s (plain ones, which stay
// in the cache, are not counted); more than one workgroup per CU drift apart
// and lose halo lines.  The shape it picks takes 1.04 times as long as the best
// one of the sweep in the geometric mean over 461 grids and forms (64-plane
// chunks and the tile height by storage form alone, 1.52 times).  Near ties go
// wrong now and then: of 6000 drawn grids and forms 0.8% take 1.02 to 1.2 times as
// long as with those, at a geometric mean of 0.52.
double march_us(const MarchForm& f, int64_t nx, int64_t ny, int64_t nz, bool fits, bool cached,
                int S, int ty, int64_t zc) {
  const double tx = static_cast<double>(ceil_div(nx, 64 * S));
  const double tyn = static_cast<double>(ceil_div(ny, ty));
  const double nch = static_cast<double>(ceil_div(nz, zc));
  const double N = static_cast<double>(nx) * static_cast<double>(ny) * static_cast<double>(nz);
  const double w = tx * tyn * nch;
  const double planes = 2.0 * static_cast<double>(ceil_div(zc + 2, 2));
  const double per_cu = std::ceil(w / f.cus);
  const double fit_lds =
      static_cast<double>(kLdsLimit / lds_bytes(f.Q, f.storage, ty, S, f.stencil));
  const double resident = std::min(per_cu, std::max(1.0, std::min(fit_lds, 32.0 / (ty + 2))));
  const double work = S * (ty + 1);
  const double full = std::floor(per_cu / resident), rest = per_cu - full * resident;
  const double lat = f.l0 + f.l1 * work, busy = f.busy * work;
  const double issue = planes * (full * std::max(lat, resident * busy) +
                                 (rest > 0 ? std::max(lat, rest * busy) : 0.0));
  double read = f.read * N * (1.0 + 2.0 * 1.5 * tyn / static_cast<double>(ny) +
                              2.0 * 2.0 * nch / static_cast<double>(nz)) +
                1.6 * 2.0 * 128.0 * f.streams * tx * static_cast<double>(ny) *
                    static_cast<double>(nz);
  if (!fits && w > f.cus && tx * tyn <= f.cus) read *= 1.1;
  const double mem = (read / 9.0 + (cached ? 0.0 : f.write * N / 5.6)) * 1e-6;
  return std::sqrt(issue * issue + mem * mem);
}

// Chunks of the shape of width_launch: at most ~512 workgroups in chunks of >=
// 64 planes, or enough workgroups in chunks of >= 8 planes.
int64_t width_zchunk(const lbfast_ctx* h) {
  const int64_t cols = ceil_div(h->p.nx, 64 * h->lane_sites) * ceil_div(h->p.ny, h->tile_rows);
  const int64_t by_blocks = std::max<int64_t>(1, 512 / cols);
  const int64_t long_chunks = std::max<int64_t>(1, h->p.nz / 64);
  if (cols * long_chunks >= 128) return ceil_div(h->p.nz, std::min(by_blocks, long_chunks));
  return ceil_div(h->p.nz, std::min(ceil_div(512, cols), std::max<int64_t>(1, h->p.nz / 8)));
}

// z-planes per workgroup of a shape, and the modelled time with them
int64_t best_zchunk(const lbfast_ctx* h, const MarchForm& f, int S, int ty, double* us) {
  const int64_t nx = h->p.nx, ny = h->p.ny, nz = h->p.nz;
  const int64_t cols = ceil_div(nx, 64 * S) * ceil_div(ny, ty);
  const bool fits = fits_cache(h);
  const bool cached = f.cached_forms && step_cached(h, S, ty);
  int64_t best = nz;
  double t_best = 0.0;
  bool have = false;
  // chunks of an even length (or one alone) leave every plane its parity; the
  // forms that keep their rows also tell the first planes of a chunk apart
  const int64_t by_width = keeps_parity(h) ? width_zchunk(h) : 0;
  const bool even_only = by_width > 0;
  const bool fixed = keeps_rows(h) || (even_only && by_width % 2 != 0 && by_width < nz);
  // in contiguous order, chunks that come out whole on each of the 8 XCDs
  // share all their halo lines there (201 x 97 x 113 D3Q27 FP32 with a field: 8
  // chunks 53 us, 9 chunks 60; over 134 in-cache grids and forms of the sweep the
  // choice is 0.4% faster for it, FP32 without a field 1.4%)
  const bool whole = !f.stencil && cache_matters(h);
  auto consider = [&](int64_t zc) {
    double t = march_us(f, nx, ny, nz, fits, cached, S, ty, zc);
    if (whole && ceil_div(nz, zc) % 8 == 0) t *= 0.95;
    if (!have || t < t_best) t_best = t, best = zc, have = true;
  };
  if (fixed) {
    consider(by_width);
  } else if (!fits && cols >= f.cus) {
    // a column for every CU: about 512 workgroups in chunks of >= 64 planes
    // (512^3 FP32: 2.00 ms, one chunk per column 2.02), FP64 with two sites
    // per lane 1024 (3.91 ms, one chunk per column 4.35; D3Q27h with one site
    // and 8 rows 4.70 ms, one chunk per column 4.07)
    const int64_t target = (f.storage == LBF_F64 && S == 2 ? 4 : 2) * int64_t{f.cus};
    const int64_t zc = ceil_div(nz, std::min(std::max<int64_t>(1, target / cols),
                                             std::max<int64_t>(1, nz / 64)));
    consider(even_only && zc < nz ? zc + zc % 2 : zc);
  } else {
    // every distinct chunk length, up to some 8 workgroups per CU
    int64_t last = 0;
    for (int64_t k = 1; k <= nz; ++k) {
      const int64_t zc = ceil_div(nz, k);
      if (zc == last) {
        k = ceil_div(nz, zc - 1) - 1;  // on to the next shorter chunk
        continue;
      }
      last = zc;
      if (k > 1 && cols * k > 8 * int64_t{f.cus}) break;
      if (!even_only || zc % 2 == 0 || zc == nz) consider(zc);
      if (zc == 1) break;
    }
  }
  if (us) *us = t_best;
  return best;
}

// Modelled time of the one-plane form, in march_us's terms: a CU's workgroups one
// after the other, `slab` busy us each, and no chain of planes before the first
// of them, against what they read (the own plane and its two neighbours, half as
// much again in the halo rows) and write, `slab_mem` bytes per site.  The step's
// constants are fitted to both forms' times on 5448 grids and forms of 10 to 300
// sites a side, states up to 120 MB: the choice takes 1.003 times as long as the
// better of the two in the geometric mean (without the memory 1.010, and 176 x
// 256 x 8 FP64 with a field 36.4 us instead of 24.4).  The adjoint's to 975 grids
// and forms, the one-plane form and a sweep of marches on each: rows, chunk and
// form together take 1.013 times as long as the best of them (1.056 with the
// states' stores left out of the march's time).
double slab_us(const lbfast_ctx* h, const MarchForm& f) {
  const double w = static_cast<double>(ceil_div(h->p.nx, 64) * ceil_div(h->p.ny, lbf::kSlabRows)) *
                   static_cast<double>(h->p.nz);
  const double issue = f.slab * f.busy * std::ceil(w / f.cus) - 1.0;
  const double mem = f.slab_mem * static_cast<double>(h->N) / 9.0 * 1e-6;
  return std::sqrt(issue * issue + mem * mem);
}

// the one-plane form in place of a march that is modelled to take `march` us
bool slab_pays(const lbfast_ctx* h, const MarchForm& f, double march) {
  return fits_cache(h) && slab_us(h, f) < march;
}

// tile shapes built for the handle's step
bool shape_built(const lbfast_ctx* h, int S, int ty) {
  if (S == 2 && h->p.nx % 2 != 0) return false;
  if (S == 3 && (h->p.nx % 3 != 0 || h->p.storage != LBF_F32 || h->p.lattice == LBF_D3Q27H ||
                 h->two_phase))
    return false;
  if (ty > 8 && (S > 1 || h->p.lattice == LBF_D3Q27H || h->two_phase)) return false;
  return lds_bytes(h->p.lattice, h->p.storage, ty, S, h->two_phase) <= kLdsLimit;
}

// The shape that explicit launch settings start from: two x-sites per lane
// where nx allows it (even, at least one 128-wide tile), 8-row tiles (FP64:
// 4 rows with two sites per lane, 6 with one) or the tallest that fits the LDS.
void width_launch(lbfast_ctx* h) {
  // two sites per lane unless 128-wide tiles would leave more of the last
  // tile empty than 64-wide ones; else three (FP32, second-order sets) where
  // 192-wide tiles leave no more empty than 64-wide ones (measured at 192^3:
  // 143 us against 178 us per step with a force field, 6-row tiles)
  const int64_t nx = h->p.nx;
  const int64_t waste1 = ceil_div(nx, 64) * 64 - nx;
  const int64_t waste2 = ceil_div(nx, 128) * 128 - nx;
  const int64_t waste3 = ceil_div(nx, 192) * 192 - nx;
  const bool three_ok = h->p.storage == LBF_F32 && h->p.lattice != LBF_D3Q27H && nx % 3 == 0 &&
                        nx >= 192 && !h->two_phase;
  if (nx % 2 == 0 && nx >= 128 && waste2 <= waste1)
    h->lane_sites = 2;
  else if (three_ok && waste3 <= waste1)
    h->lane_sites = 3;
  else
    h->lane_sites = 1;
  // D3Q27h spills registers with two sites per lane in FP64.  The 16-bit forms
  // keep two since their planes are grouped (measured at 512^3, one / two
  // sites: FP16 65.9 / 68.0 GLUPS, split FP16 61.0 / 67.1, BF16 70.0 / 70.2)
  if (h->p.lattice == LBF_D3Q27H && h->p.storage == LBF_F64) h->lane_sites = 1;
  h->tile_rows = 4;
  const bool f64 = h->p.storage == LBF_F64;
  const int first = f64 ? (h->lane_sites == 2 ? 4 : 6) : (h->lane_sites == 3 ? 6 : 8);
  for (int ty : {first, 6, 4})
    if (lds_bytes(h->p.lattice, h->p.storage, ty, h->lane_sites) <= kLdsLimit) {
      h->tile_rows = ty;
      break;
    }
  h->z_chunk = 0;
}

// Default launch shape: the one of the least modelled time among those built,
// but
//   * 16-bit storage keeps the sites per lane that the width alone gives:
//     the one- and two-site kernels contract FP32 differently, which shows in 2%
//     of the stored 16-bit words after ten steps, and a run's values should not
//     depend on the other extents (see keeps_parity for what else it keeps);
//   * FP64: one site per lane for D3Q27 and D3Q27h (two spill or leave one
//     short workgroup per CU), and two sites where the width suits them, with
//     4 rows, for D3Q19 beyond the cache (256^3: 497 us, 6 rows 575, one site
//     and 14 rows 637) and for D3Q27 without a force field with a column for
//     every CU (512^3 3.78 ms, one site and 8 rows 3.95; 256^3 0.545, 0.530);
//   * variable density or viscosity: one site per lane (two spill; 256^3 FP32
//     0.80 ms against 0.57);
//   * 6 rows at most with three sites (8 spill with a force field: 192^3 143 us
//     against 199), for the two-component step with D3Q27 and D3Q27h with two
//     sites or FP64 (256^3 FP32 645 us with two sites and 8 rows, 542 with one;
//     192^3 FP64 938 us with 8 rows, 654 with 6), and for D3Q27h FP64 with a
//     force field (8 spill: 130^3 181 us, 144 with 6).  With a uniform force
//     instead, 8 rows spill 20 to 32 bytes and are as fast or faster (130^3 124
//     and 137 us, 256^3 608 and 664, 192^3 302 and 281), and the two-site form of
//     D3Q27, 44 to 80 bytes, is faster on some of the grids that take it and
//     slower on others (384 x 384 x 256 1473 us, one site 1638; 512 x 512 x 300 2621
//     and 2371).
void model_launch(lbfast_ctx* h) {
  const int64_t nx = h->p.nx;
  const bool f64 = h->p.storage == LBF_F64;
  const bool two = nx % 2 == 0 && nx >= 128 &&
                   ceil_div(nx, 128) * 128 - nx <= ceil_div(nx, 64) * 64 - nx;
  const bool wide27 = f64 && h->p.lattice == LBF_D3Q27 && two && !h->Ffield && !h->two_phase &&
                      !fits_cache(h) && ceil_div(nx, 128) * ceil_div(h->p.ny, 4) >= h->cus;
  const bool one_only = (h->two_phase && variable_properties(h)) ||
                        (f64 && h->p.lattice != LBF_D3Q19 && !wide27);
  h->auto_slab = false;
  if (keeps_rows(h)) {
    h->auto_sites = h->lane_sites;
    h->auto_rows = h->tile_rows;
    return;
  }
  const MarchForm f = march_form(h);
  double t_best = 0.0;
  bool have = false;
  for (int S = 1; S <= 3; ++S) {
    if (one_only && S != 1) continue;
    if (is_16bit(h->p.storage) && !one_only && S != (two ? 2 : 1)) continue;
    for (int ty : lbf::kTileRowsSupported) {
      if (!shape_built(h, S, ty)) continue;
      if (ty > 6 && (S == 3 || (h->two_phase && h->p.lattice != LBF_D3Q19 && (S == 2 || f64)) ||
                     (f64 && h->p.lattice == LBF_D3Q27H && h->Ffield)))
        continue;
      if (f64 && !one_only && !fits_cache(h) && (two ? (S != 2 || ty != 4) : S != 1)) continue;
      double t;
      (void)best_zchunk(h, f, S, ty, &t);
      if (!have || t < t_best) {
        have = true;
        t_best = t;
        h->auto_sites = S;
        h->auto_rows = ty;
      }
    }
  }
  // not 16-bit storage: with a uniform force the one-plane form is contracted
  // differently (FP16 D3Q19 33 x 70 x 40: some words off by one after 3 steps)
  h->auto_slab = !is_16bit(h->p.storage) && slab_pays(h, f, t_best);
}

bool step_slab(const lbfast_ctx* h) {
  if (h->form != LBF_FORM_AUTO) return h->form == LBF_FORM_ONE_PLANE;
  return !h->shape_set && h->z_chunk == 0 && h->auto_slab;
}

// launch geometry of the one-plane form
Launch slab_launch(const lbfast_ctx* h) {
  Launch l{};
  l.slab = 1;
  l.lane_sites = 1;
  l.rows = lbf::kSlabRows;
  l.tiles_x = static_cast<int>(ceil_div(h->p.nx, 64));
  l.tiles_y = static_cast<int>(ceil_div(h->p.ny, lbf::kSlabRows));
  l.zchunk = 1;
  l.zchunks = static_cast<int>(h->p.nz);
  // z-neighbours on one XCD once a CU has more than one workgroup (48^3 FP32
  // 5.7 us, 7.7 in the hardware's order; 32^3 4.1 and 3.8)
  l.xcd_remap = h->block_order != 0
                    ? h->block_order == 2
                    : static_cast<int64_t>(l.tiles_x) * l.tiles_y * h->p.nz > h->cus;
  return l;
}

int step_sites(const lbfast_ctx* h) { return h->shape_set ? h->lane_sites : h->auto_sites; }
int step_rows(const lbfast_ctx* h) { return h->shape_set ? h->tile_rows : h->auto_rows; }

// tiles and z-chunks of a march of the given shape
Launch march_launch(const lbfast_ctx* h, const MarchForm& f, int lane_sites, int rows) {
  Launch l{};
  l.lane_sites = lane_sites;
  l.rows = rows;
  l.tiles_x = static_cast<int>(ceil_div(h->p.nx, 64 * lane_sites));
  l.tiles_y = static_cast<int>(ceil_div(h->p.ny, rows));
  int64_t zc = h->z_chunk;
  if (zc <= 0) zc = best_zchunk(h, f, lane_sites, rows, nullptr);
  if (zc > h->p.nz) zc = h->p.nz;
  l.zchunk = static_cast<int>(zc);
  l.zchunks = static_cast<int>(ceil_div(h->p.nz, zc));
  return l;
}

// Rows per tile of the adjoint step: 8 (FP64: 6, taller tiles spill), or fewer
// where the states fit the cache and the model says so (FP32 16^3 to 48^3
// 4 or 6 rows 11.5 to 12.5 us per step against 12.8 to 15.2).
int adjoint_rows(const lbfast_ctx* h, const MarchForm& f, int sites) {
  if (h->adj_rows) return h->adj_rows;
  const int most = h->p.storage == LBF_F64 ? 6 : 8;
  if (sites != 1 || !fits_cache(h)) return most;
  int best = most;
  double t_best = 0.0;
  for (int ty : {most, 6, 4}) {
    double t;
    (void)best_zchunk(h, f, sites, ty, &t);
    if (ty == most || t < t_best) t_best = t, best = ty;
  }
  return best;
}

// Block order: a contiguous range of tiles per XCD where the state is in the
// cache and large enough for its halo lines to matter (201 x 97 x 113 FP32
// 38 us against 47 in the hardware's order; 64^3 10.0 against 9.0).  Beyond the
// cache for the FP64 step of D3Q19 (13 grids from 180 x 250 x 120 to 320^3 4%
// faster, with a force field too: 256^3 481 us against 537, 250^3 506 and 531,
// 320^3 1013 and 1035; 275 x 245 x 97 4% slower), and otherwise in FP64 with
// more columns than CUs (512^3 D3Q19 3.91 ms against 5.55; with fewer columns
// D3Q27 and D3Q27h are as fast in either on 13 grids, but 320^3 1313 us against
// 1115).  Elsewhere the hardware's order: marches of one wave of workgroups keep
// step by themselves, and several waves lose about 10% in the other.  The
// two-component step is no exception: on 52 grids and forms in the cache the
// contiguous order takes 0.94 times as long in the geometric mean (180 x 90 x 60
// FP32 51.8 us per step of both passes against 75, 201 x 97 x 113 125 against
// 145; at most 1.2% slower), and for FP64 D3Q19 beyond it 0.97 (128^3 140 and 153,
// 256^3 969 and 1001), but not with contrast there (equal on six grids, 256 x 300
// x 180 976 and 877).
bool contiguous_order(const lbfast_ctx* h, int tiles_x, int tiles_y, bool adjoint = false) {
  if (h->block_order != 0) return h->block_order == 2;
  // measured 6% slower for 16-bit D3Q27h at 267 x 122 x 127
  if (keeps_rows(h)) return false;
  if (fits_cache(h)) return cache_matters(h);
  if (h->two_phase && variable_properties(h)) return false;
  return h->p.storage == LBF_F64 && ((h->p.lattice == LBF_D3Q19 && !adjoint) ||
                                     static_cast<int64_t>(tiles_x) * tiles_y > h->cus);
}

// The launches that the handle's settings come to; whatever changes one of them
// (the set_ calls, the force field, the two-component variant) calls this.
void plan(lbfast_ctx* h) {
  if (step_slab(h)) {
    h->step = slab_launch(h);
  } else {
    const int sites = step_sites(h), rows = step_rows(h);
    h->step = march_launch(h, march_form(h), sites, rows);
    h->step.cached = step_cached(h, sites, rows);
    h->step.xcd_remap = contiguous_order(h, h->step.tiles_x, h->step.tiles_y);
  }
  if (h->two_phase) {
    const int nx = static_cast<int>(h->p.nx), ny = static_cast<int>(h->p.ny);
    const int nz = static_cast<int>(h->p.nz);
    h->phase = lbf::phase_geom(h->p.storage, nx, ny, nz, h->cus);
    h->force = lbf::force_geom(h->p.storage, h->pp.rho_l != h->pp.rho_h, nx, ny, nz, h->cus);
  }
}

// problem and default launch shapes of a new handle
void set_params(lbfast_ctx* h, const lbfast_params* p) {
  h->p = *p;
  h->N = p->nx * p->ny * p->nz;
  width_launch(h);
  model_launch(h);
  plan(h);
}

// The shapes of a handle that has become a two-component one.
void two_phase_launch(lbfast_ctx* h) {
  // A shape chosen by the caller is kept where it can be.  The two-component
  // step has one- and two-site forms of at most 8 rows,
  // with one more LDS slot (phi(t+1)) than the one-component step.  With
  // variable density or viscosity, one site per lane: the two-site form
  // spills registers there (measured at 256^3 FP32: 0.80 ms against 0.57).
  const bool one_site = h->lane_sites == 3 || (h->lane_sites == 2 && variable_properties(h));
  const bool reshape = one_site || h->tile_rows > 8 ||
                       lds_bytes(h->p.lattice, h->p.storage, h->tile_rows, h->lane_sites,
                                 true) > kLdsLimit;
  if (one_site) h->lane_sites = 1;
  if (reshape) {
    h->tile_rows = 4;
    for (int ty : {8, 6})
      if (lds_bytes(h->p.lattice, h->p.storage, ty, h->lane_sites, true) <= kLdsLimit) {
        h->tile_rows = ty;
        break;
      }
  }
  model_launch(h);
  plan(h);
}

int check_handle(lbfast_t h) {
  if (!h) return fail(LBF_E_ARG, "handle is NULL");
  return LBF_OK;
}

struct DeviceGuard {
  int prev = -1;
  explicit DeviceGuard(int dev) {
    if (hipGetDevice(&prev) != hipSuccess) prev = -1;
    if (prev != dev) (void)hipSetDevice(dev);
  }
  ~DeviceGuard() {
    int now;
    if (prev >= 0 && hipGetDevice(&now) == hipSuccess && now != prev) (void)hipSetDevice(prev);
  }
};

bool is_device_ptr(const void* p) {
  hipPointerAttribute_t at;
  if (hipPointerGetAttributes(&at, p) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  return at.type == hipMemoryTypeDevice || at.type == hipMemoryTypeManaged;
}

// whether two arrays share memory (nullptr: no array)
bool overlap(const void* a, size_t na, const void* b, size_t nb) {
  const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
  return a && b && x < y + nb && y < x + na;
}

int set_geometry(const Launch& l, lbf::StepArgs* a) {
  if (static_cast<int64_t>(l.tiles_x) * l.tiles_y * l.zchunks > 0x7fffffff)
    return fail(LBF_E_ARG, "grid too large");
  a->slab = l.slab;
  a->cached = l.cached;
  a->xcd_remap = l.xcd_remap;
  a->lane_sites = l.lane_sites;
  a->tiles_x = l.tiles_x;
  a->tiles_y = l.tiles_y;
  a->zchunk = l.zchunk;
  a->zchunks = l.zchunks;
  return LBF_OK;
}

// launch geometry, relaxation, force and scales of the handle's step
int step_args(const lbfast_ctx* h, lbf::StepArgs* a) {
  *a = lbf::StepArgs{};
  a->nx = static_cast<int>(h->p.nx);
  a->ny = static_cast<int>(h->p.ny);
  a->nz = static_cast<int>(h->p.nz);
  a->N = h->N;
  if (int rc = set_geometry(h->step, a)) return rc;
  a->omega = 1.0 / h->p.tau;
  for (int k = 0; k < 3; ++k) a->F[k] = h->Ffield ? 0.0 : h->p.force[k];
  for (int k = 0; k < 10; ++k) {
    a->scale[k] = h->scale[k];
    a->inv_scale[k] = h->inv_scale[k];
  }
  {
    const double inv_d = 1.0 / ((h->p.lattice == LBF_D3Q19) ? 9.0 : 27.0);
    const float hi = static_cast<float>(inv_d);
    const float lo = static_cast<float>(inv_d - static_cast<double>(hi));
    for (int k = 0; k < 4; ++k) {
      a->enc_hi[k] = hi * h->inv_scale[k];
      a->enc_lo[k] = lo * h->inv_scale[k];
    }
  }
  a->Ffield = h->Ffield;
  a->stochastic = h->p.rounding == LBF_ROUND_STOCHASTIC ||
                  (h->p.rounding == LBF_ROUND_AUTO && h->p.storage == LBF_BF16S);
  if (h->two_phase) {
    // the phases' relaxation times replace params.tau
    a->omega = 1.0 / h->pp.tau_l;
    a->rho_l = h->pp.rho_l;
    a->rho_h = h->pp.rho_h;
    a->nu_l = (h->pp.tau_l - 0.5) / 3.0;
    a->nu_h = (h->pp.tau_h - 0.5) / 3.0;
  }
  return LBF_OK;
}

// Launch geometry of the adjoint step, which reads 22 values per destination
// site: by default one site per lane and 8-row tiles (FP64: 6);
// lbfast_set_adjoint_launch may choose two or three sites per lane with 4- or
// 6-row tiles (FP32).
Launch adjoint_launch(const lbfast_ctx* h) {
  if (h->form == LBF_FORM_ONE_PLANE) return slab_launch(h);
  const MarchForm f = march_form(h, true);
  const int sites = h->adj_sites ? h->adj_sites : 1;
  const int rows = adjoint_rows(h, f, sites);
  if (h->form == LBF_FORM_AUTO && !h->adj_sites && !h->adj_rows && h->z_chunk == 0) {
    double march;
    (void)best_zchunk(h, f, sites, rows, &march);
    if (slab_pays(h, f, march)) return slab_launch(h);
  }
  Launch l = march_launch(h, f, sites, rows);
  l.xcd_remap = contiguous_order(h, l.tiles_x, l.tiles_y, true);
  return l;
}

// seed of the stochastic rounding of step t (16-bit storage): the step
// counter through SplitMix64's output mix (Steele, Lea and Flood, 2014), so
// that every step draws fresh bits per site
uint32_t step_seed(uint64_t t) {
  uint64_t x = t + 0x9E3779B97F4A7C15ull;
  x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
  x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
  return static_cast<uint32_t>(x ^ (x >> 31));
}

int launch_forward(const lbfast_ctx* h, const lbf::StepArgs& a) {
  hipError_t e = lbf::launch_step(h->p.lattice, h->p.storage, h->step.rows,
                                  h->p.bc[1] == LBF_WALLS, a, h->stream);
  if (e != hipSuccess) return hip_fail(e, "step launch");
  return LBF_OK;
}

size_t compute_bytes(const lbfast_ctx* h) { return h->p.storage == LBF_F64 ? 8 : 4; }

// phase-field launch arguments for the current time level
lbf::PhaseArgs phase_args(const lbfast_ctx* h) {
  lbf::PhaseArgs a{};
  a.phi = h->phi[h->pcur];
  a.phi_out = h->phi[h->pcur ^ 1];
  a.state = h->buf[h->cur];
  a.F = h->Fph[h->pcur ^ 1];
  a.nx = static_cast<int>(h->p.nx);
  a.ny = static_cast<int>(h->p.ny);
  a.nz = static_cast<int>(h->p.nz);
  a.N = h->N;
  a.D = h->pp.diffusivity;
  a.lambda = 4.0 * h->pp.diffusivity / h->pp.width;
  a.beta = 12.0 * h->pp.sigma / h->pp.width;
  a.kappa = 1.5 * h->pp.sigma * h->pp.width;
  a.eps = 1e-12;  // n = grad(phi) / (|grad(phi)| + eps)
  for (int k = 0; k < 3; ++k) a.Fb[k] = h->p.force[k];  // body acceleration
  for (int k = 0; k < 10; ++k) a.scale[k] = h->scale[k];
  a.walls_y = h->p.bc[1] == LBF_WALLS;
  a.contrast = h->pp.rho_l != h->pp.rho_h;
  a.rho_l = h->pp.rho_l;
  a.rho_h = h->pp.rho_h;
  a.nu_l = (h->pp.tau_l - 0.5) / 3.0;
  a.nu_h = (h->pp.tau_h - 0.5) / 3.0;
  return a;
}

int check_adjoint_args(const lbfast_ctx* h, int64_t nsteps, int64_t every) {
  if (h->two_phase)
    return fail(LBF_E_UNSUPPORTED, "the adjoint does not cover the two-component variant");
  if (h->p.storage != LBF_F64 && h->p.storage != LBF_F32)
    return fail(LBF_E_UNSUPPORTED, "the adjoint supports F64 and F32 storage only");
  if (h->p.lattice == LBF_D3Q27H)
    return fail(LBF_E_UNSUPPORTED, "the adjoint covers the second-order sets D3Q19 and D3Q27");
  if (nsteps < 0) return fail(LBF_E_ARG, "nsteps must be >= 0");
  if (every < 1) return fail(LBF_E_ARG, "every must be >= 1");
  return LBF_OK;
}

}  // namespace

extern "C" {

int lbfast_abi_version(void) { return LBFAST_ABI_VERSION; }

size_t lbfast_buffer_bytes(const lbfast_params* p) {
  if (validate(p) != LBF_OK) return 0;
  return static_cast<size_t>(p->nx) * static_cast<size_t>(p->ny) * static_cast<size_t>(p->nz) *
         state_planes(p->storage) * elem_bytes(p->storage);
}

const char* lbfast_last_error(void) { return g_err.c_str(); }

int lbfast_stream_probe(const void* src, void* dst, int64_t n, int nplanes, void* stream) {
  g_err.clear();
  if (!src || !dst) return fail(LBF_E_ARG, "null buffer");
  if (n < 1 || static_cast<double>(n) * 4.0 >= 4294967296.0)
    return fail(LBF_E_ARG, "n must be in [1, 2^30)");
  if (nplanes < 1) return fail(LBF_E_ARG, "nplanes must be >= 1");
  hipError_t e = lbf::launch_stream_probe(src, dst, n, nplanes, static_cast<hipStream_t>(stream));
  if (e != hipSuccess) return hip_fail(e, "stream probe");
  return LBF_OK;
}

int lbfast_copy_probe(const void* src, void* dst, int64_t n4, void* stream) {
  g_err.clear();
  if (!src || !dst) return fail(LBF_E_ARG, "null buffer");
  if ((reinterpret_cast<uintptr_t>(src) | reinterpret_cast<uintptr_t>(dst)) & 15)
    return fail(LBF_E_ARG, "buffers must be 16-byte aligned");
  if (n4 < 1) return fail(LBF_E_ARG, "n4 must be >= 1");
  hipError_t e = lbf::launch_copy_probe(src, dst, n4, static_cast<hipStream_t>(stream));
  if (e != hipSuccess) return hip_fail(e, "copy probe");
  return LBF_OK;
}

int lbfast_planes_probe(const void* src, void* dst, int64_t n, int nplanes, void* stream) {
  g_err.clear();
  if (!src || !dst) return fail(LBF_E_ARG, "null buffer");
  if ((reinterpret_cast<uintptr_t>(src) | reinterpret_cast<uintptr_t>(dst)) & 7)
    return fail(LBF_E_ARG, "buffers must be 8-byte aligned");
  if (n < 2 || n % 2) return fail(LBF_E_ARG, "n must be even and >= 2");
  if (nplanes < 1 || nplanes > 10) return fail(LBF_E_ARG, "nplanes must be in [1, 10]");
  hipError_t e = lbf::launch_planes_probe(src, dst, n, nplanes, static_cast<hipStream_t>(stream));
  if (e != hipSuccess) return hip_fail(e, "planes probe");
  return LBF_OK;
}

int lbfast_zmarch_probe(const void* src, void* dst, int nx, int ny, int nz, int layout,
                        int zchunk, void* stream) {
  g_err.clear();
  if (!src || !dst) return fail(LBF_E_ARG, "null buffer");
  if ((reinterpret_cast<uintptr_t>(src) | reinterpret_cast<uintptr_t>(dst)) & 15)
    return fail(LBF_E_ARG, "buffers must be 16-byte aligned");
  if (nx < 128 || nx % 128) return fail(LBF_E_ARG, "nx must be a positive multiple of 128");
  if (ny < 8 || ny % 8) return fail(LBF_E_ARG, "ny must be a positive multiple of 8");
  if (nz < 1 || zchunk < 1) return fail(LBF_E_ARG, "nz and zchunk must be >= 1");
  if (layout < 0 || layout > 3) return fail(LBF_E_ARG, "layout must be in [0, 3]");
  if (static_cast<int64_t>(nx / 128) * (ny / 8) * ((nz + zchunk - 1) / zchunk) > 0x7fffffff)
    return fail(LBF_E_ARG, "grid too large");
  hipError_t e = lbf::launch_zmarch_probe(src, dst, nx, ny, nz, layout, zchunk,
                                          static_cast<hipStream_t>(stream));
  if (e != hipSuccess) return hip_fail(e, "z-march probe");
  return LBF_OK;
}

int lbfast_create(const lbfast_params* p, void* stream, void* buf0, void* buf1, lbfast_t* out) {
  g_err.clear();
  if (!out) return fail(LBF_E_ARG, "out is NULL");
  *out = nullptr;
  int rc = validate(p);
  if (rc != LBF_OK) return rc;
  if ((buf0 == nullptr) != (buf1 == nullptr))
    return fail(LBF_E_ARG, "pass both buffers or neither");
  if (buf0 && buf0 == buf1) return fail(LBF_E_ARG, "buf0 and buf1 must differ");
  if ((buf0 && (reinterpret_cast<uintptr_t>(buf0) & 255)) ||
      (buf1 && (reinterpret_cast<uintptr_t>(buf1) & 255)))
    return fail(LBF_E_ARG, "buffers must be 256-byte aligned");

  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_fail(e, "hipGetDevice");

  lbfast_ctx* h = new (std::nothrow) lbfast_ctx();
  if (!h) return fail(LBF_E_NOMEM, "host allocation failed");
  h->device = dev;
  int cus = 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess &&
      cus > 0)
    h->cus = cus;
  else
    (void)hipGetLastError();
  set_params(h, p);
  h->stream = static_cast<hipStream_t>(stream);
  const size_t bytes = lbfast_buffer_bytes(p);
  for (int k = 0; k < 10; ++k) {
    h->scale[k] = (p->scale[k] != 0.0f) ? p->scale[k] : 1.0f;
    h->inv_scale[k] = 1.0f / h->scale[k];
  }
  const bool s16 = is_16bit(p->storage);
  h->scales_fixed = !s16;
  if (s16) {
    bool all = true;
    for (int k = 0; k < 10; ++k) all = all && p->scale[k] != 0.0f;
    h->scales_fixed = all;
  }
  if (buf0) {
    h->buf[0] = buf0;
    h->buf[1] = buf1;
    h->owned = false;
  } else {
    h->owned = true;
    for (int i = 0; i < 2; ++i) {
      e = hipMalloc(&h->buf[i], bytes);
      if (e != hipSuccess) {
        (void)hipGetLastError();
        if (h->buf[0]) (void)hipFree(h->buf[0]);
        delete h;
        return fail(LBF_E_NOMEM, "hipMalloc of %zu bytes failed", bytes);
      }
    }
  }
  e = hipMalloc(reinterpret_cast<void**>(&h->d_partials),
                (lbf::kReduceBlocks * 5 + 5) * sizeof(double));
  if (e == hipSuccess) e = hipMalloc(reinterpret_cast<void**>(&h->d_maxbits), 16 * sizeof(unsigned));
  if (e == hipSuccess) e = hipMemsetAsync(h->buf[0], 0, bytes, h->stream);
  if (e == hipSuccess) e = hipMemsetAsync(h->buf[1], 0, bytes, h->stream);
  if (e != hipSuccess) {
    int r = hip_fail(e, "create");
    lbfast_destroy(h);
    return r;
  }
  *out = h;
  return LBF_OK;
}

int lbfast_destroy(lbfast_t h) {
  if (!h) return LBF_OK;
  DeviceGuard g(h->device);
  if (h->stream) (void)hipStreamSynchronize(h->stream);
  else (void)hipDeviceSynchronize();
  if (h->owned) {
    if (h->buf[0]) (void)hipFree(h->buf[0]);
    if (h->buf[1]) (void)hipFree(h->buf[1]);
  }
  for (void* p : {h->phi[0], h->phi[1], h->Fph[0], h->Fph[1]})
    if (p) (void)hipFree(p);
  if (h->d_partials) (void)hipFree(h->d_partials);
  if (h->d_maxbits) (void)hipFree(h->d_maxbits);
  delete h;
  return LBF_OK;
}

int lbfast_set_moments(lbfast_t h, const void* m, int dtype, int on_device) {
  g_err.clear();
  if (int rc = check_handle(h)) return rc;
  if (!m) return fail(LBF_E_ARG, "moment array is NULL");
  if (dtype != LBF_F64 && dtype != LBF_F32) return fail(LBF_E_ARG, "dtype must be F64 or F32");
  if (on_device != 0 && on_device != 1) return fail(LBF_E_ARG, "on_device must be 0 or 1");
  DeviceGuard g(h->device);
  const size_t ub = (dtype == LBF_F64) ? 8 : 4;
  const int64_t N = h->N;
  const size_t pbytes = static_cast<size_t>(N) * ub;
  hipError_t e = hipSuccess;
  // Device input is read in place.  Host input goes through a device staging
  // area: the three velocity planes (kept for the whole call, the deviation
  // storage of the second-order planes needs them) and one plane at a time.
  char* staging = nullptr;
  if (!on_device) {
    e = hipMalloc(reinterpret_cast<void**>(&staging), 4 * pbytes);
    if (e != hipSuccess) {
      (void)hipGetLastError();
      return fail(LBF_E_NOMEM, "staging allocation failed");
    }
    e = hipMemcpyAsync(staging, static_cast<const char*>(m) + pbytes, 3 * pbytes,
                       hipMemcpyHostToDevice, h->stream);
  }
  const void* u[3];
  for (int c = 0; c < 3; ++c)
    u[c] = on_device ? static_cast<const char*>(m) + (1 + c) * pbytes
                     : static_cast<const void*>(staging + c * pbytes);
  // device pointer of user plane k (host planes are copied in first)
  auto plane = [&](int k, hipError_t& err) -> const void* {
    if (on_device) return static_cast<const char*>(m) + k * pbytes;
    if (k >= 1 && k <= 3) return staging + (k - 1) * pbytes;
    char* p = staging + 3 * pbytes;
    err = hipMemcpyAsync(p, static_cast<const char*>(m) + k * pbytes, pbytes,
                         hipMemcpyHostToDevice, h->stream);
    return p;
  };
  // automatic 16-bit scales: the power of two placing the magnitude M of the
  // plane's group just below 2^10, which leaves a factor 64 of growth before
  // FP16 overflows (65504); FP16 keeps its relative precision down to 2^-14.
  // M is max|u| for the velocity planes, max(|a2|, max|u|^2) for the
  // second-order planes and max(|p*|, 3 max|u|^2) for p*: a plane that starts
  // at zero (p* of a solenoidal field, u_z of a planar flow) takes its group's
  // magnitude instead of a scale of 1, which would put its later values in
  // FP16's subnormal range.
  if (!h->scales_fixed) {
    float mx[10] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    for (int pass = 0; pass < 2 && e == hipSuccess; ++pass) {
      const int k0 = pass == 0 ? 0 : 4, k1 = pass == 0 ? 4 : 10;
      e = hipMemsetAsync(h->d_maxbits, 0, 16 * sizeof(unsigned), h->stream);
      for (int k = k0; k < k1 && e == hipSuccess; ++k) {
        const void* src = plane(k, e);
        if (e == hipSuccess)
          e = lbf::launch_maxabs(h->p.storage, dtype, src, u, N, k, h->inv_scale, h->scale,
                                 h->d_maxbits, h->stream);
        // the single plane slot of the staging area is reused: wait before the next copy
        if (e == hipSuccess && !on_device) e = hipStreamSynchronize(h->stream);
      }
      unsigned bits[16];
      if (e == hipSuccess)
        e = hipMemcpyAsync(bits, h->d_maxbits, sizeof bits, hipMemcpyDeviceToHost, h->stream);
      if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
      if (e != hipSuccess) break;
      for (int k = k0; k < k1; ++k) {
        std::memcpy(&mx[k], &bits[k], sizeof(float));
        if (!std::isfinite(mx[k])) mx[k] = 0.0f;
      }
    }
    if (e == hipSuccess) {
      const float um = std::max(mx[1], std::max(mx[2], mx[3]));
      float am = um * um;
      for (int k = 4; k < 10; ++k) am = std::max(am, mx[k]);
      const float pm = std::max(mx[0], 3.0f * um * um);
      for (int k = 0; k < 10; ++k) {
        if (h->p.scale[k] != 0.0f) continue;
        const float M = k == 0 ? pm : (k < 4 ? um : am);
        float sc = 1.0f;
        if (M > 0.0f) {
          int ex;
          std::frexp(M, &ex);              // M in [2^(ex-1), 2^ex)
          sc = std::ldexp(1.0f, ex - 10);  // M / sc < 2^10
        }
        h->scale[k] = sc;
        h->inv_scale[k] = 1.0f / sc;
      }
      h->scales_fixed = true;
    }
  }
  void* dst = h->buf[h->cur];
  // device arrays in one pass (the vector accesses want 16-byte alignment)
  const bool whole = on_device && reinterpret_cast<uintptr_t>(m) % 16 == 0 &&
                     lbf::whole_state_blocks(h->p.storage, dtype, false, N) > 0;
  if (whole && e == hipSuccess)
    e = lbf::launch_encode_all(h->p.storage, dtype, m, dst, N, h->inv_scale, h->scale, h->stream);
  for (int k = 0; k < 10 && e == hipSuccess && !whole; ++k) {
    const void* src = plane(k, e);
    if (e == hipSuccess)
      e = lbf::launch_encode(h->p.storage, dtype, src, u, dst, N, k, h->inv_scale, h->scale,
                             h->stream);
    if (e == hipSuccess && !on_device) e = hipStreamSynchronize(h->stream);
  }
  if (staging) {
    hipError_t e2 = hipStreamSynchronize(h->stream);
    if (e == hipSuccess) e = e2;
    (void)hipFree(staging);
  }
  if (e != hipSuccess) return hip_fail(e, "set_moments");
  return LBF_OK;
}

int lbfast_get_moments(lbfast_t h, void* m, int dtype, int on_device) {
  g_err.clear();
  if (int rc = check_handle(h)) return rc;
  if (!m) return fail(LBF_E_ARG, "moment array is NULL");
  if (dtype != LBF_F64 && dtype != LBF_F32) return fail(LBF_E_ARG, "dtype must be F64 or F32");
  if (on_device != 0 && on_device != 1) return fail(LBF_E_ARG, "on_device must be 0 or 1");
  DeviceGuard g(h->device);
  const size_t ub = (dtype == LBF_F64) ? 8 : 4;
  const int64_t N = h->N;
  const size_t pbytes = static_cast<size_t>(N) * ub;
  const void* src = h->buf[h->cur];
  hipError_t e = hipSuccess;
  void* staging = nullptr;
  if (!on_device) {
    e = hipMalloc(&staging, pbytes);
    if (e != hipSuccess) {
      (void)hipGetLastError();
      return fail(LBF_E_NOMEM, "staging allocation failed");
    }
  }
  const bool whole = on_device && reinterpret_cast<uintptr_t>(m) % 16 == 0 &&
                     lbf::whole_state_blocks(h->p.storage, dtype, true, N) > 0;
  if (whole) e = lbf::launch_decode_all(h->p.storage, dtype, src, m, N, h->scale, h->stream);
  for (int k = 0; k < 10 && e == hipSuccess && !whole; ++k) {
    void* dst = on_device ? static_cast<void*>(static_cast<char*>(m) + k * pbytes) : staging;
    e = lbf::launch_decode(h->p.storage, dtype, src, dst, N, k, h->scale, h->stream);
    if (e == hipSuccess && !on_device)
      e = hipMemcpyAsync(static_cast<char*>(m) + k * pbytes, staging, pbytes,
                         hipMemcpyDeviceToHost, h->stream);
    if (e == hipSuccess && !on_device) e = hipStreamSynchronize(h->stream);
  }
  if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
  if (staging) (void)hipFree(staging);
  if (e != hipSuccess) return hip_fail(e, "get_moments");
  return LBF_OK;
}

int lbfast_set_force_field(lbfast_t h, const void* F_dev, int dtype) {
  g_err.clear();
  if (int rc = check_handle(h)) return rc;
  if (h->two_phase)
    return fail(LBF_E_STATE, "the two-component variant computes its own force field");
  if (!F_dev) {
    const bool had = h->Ffield != nullptr;
    h->Ffield = nullptr;
    if (had) {
      model_launch(h);
      plan(h);
    }
    return LBF_OK;
  }
  const int want = (h->p.storage == LBF_F64) ? LBF_F64 : LBF_F32;
  if (dtype != want)
    return fail(LBF_E_ARG, "force field dtype must be the compute type (%s)",
                want == LBF_F64 ? "F64" : "F32");
  if (reinterpret_cast<uintptr_t>(F_dev) & (dtype == LBF_F64 ? 7 : 3))
    return fail(LBF_E_ARG, "force field is misaligned");
  if (!is_device_ptr(F_dev)) return fail(LBF_E_ARG, "force field must be device memory");
  const bool had = h->Ffield != nullptr;
  h->Ffield = F_dev;
  if (!had) {
    model_launch(h);
    plan(h);
  }
  return LBF_OK;
}

int lbfast_set_launch(lbfast_t h, int tile_rows, int z_chunk) {
  g_err.clear();
  if (int rc = check_handle(h)) return rc;
  if (tile_rows != 0) {
    bool ok = false;
    for (int t : lbf::kTileRowsSupported) ok = ok || t == tile_rows;
    if (!ok) return fail(LBF_E_ARG, "tile_rows %d not supported (4, 6, 8 or 14)", tile_rows);
    if (h->lane_sites >= 2 && tile_rows > 8)
      return fail(LBF_E_UNSUPPORTED, "two or three x-sites per lane support tiles of at most 8 rows");
    if (h->p.lattice == LBF_D3Q27H && tile_rows > 8)
      return fail(LBF_E_UNSUPPORTED, "D3Q27h supports tiles of at most 8 rows");
    const size_t lb = lds_bytes(h->p.lattice, h->p.storage, tile_rows, h->lane_sites, h->two_phase);
    if (lb > kLdsLimit)
      return fail(LBF_E_UNSUPPORTED, "tile_rows %d needs %zu bytes of LDS (limit 160 KiB)",
                  tile_rows, lb);
  }
  if (z_chunk < 0) return fail(LBF_E_ARG, "z_chunk must be >= 0");
  if (tile_rows) {
    h->tile_rows = tile_rows;
    h->shape_set = true;
  }
  if (z_chunk) h->z_chunk = z_chunk;
  plan(h);
  return LBF_OK;
}

int lbfast_set_block_order(lbfast_t h, int order) {
  g_err.clear();
  if (int rc = check_handle(h)) return rc;
  if (order < 0 || order > 2) return fail(LBF_E_ARG, "order must be 0, 1 or 2");
  h->block_order = order;
  plan(h);
  return LBF_OK;
}

int lbfast_set_lane_sites(lbfast_t h, int sites) {
  g_err.clear();
  if (int rc = check_handle(h)) return rc;
  if (sites != 1 && sites != 2 && sites != 3) return fail(LBF_E_ARG, "sites must be 1, 2 or 3");
  if (sites == 2 && h->p.nx % 2 != 0)
    return fail(LBF_E_UNSUPPORTED, "two x-sites per lane need an even nx");
  if (sites == 3 && (h->p.nx % 3 != 0 || h->p.storage != LBF_F32 ||
                     h->p.lattice == LBF_D3Q27H || h->two_phase))
    return fail(LBF_E_UNSUPPORTED,
                "three x-sites per lane need nx divisible by 3, F32 storage, a second-order "
                "set and one component");
  // keep the tile height if it fits, else the tallest one (of 8, 6, 4) that does
  int ty = h->tile_rows;
  if ((sites >= 2 && ty > 8) ||
      lds_bytes(h->p.lattice, h->p.storage, ty, sites, h->two_phase) > kLdsLimit) {
    ty = 0;
    for (int t : {8, 6, 4})
      if (lds_bytes(h->p.lattice, h->p.storage, t, sites, h->two_phase) <= kLdsLimit) {
        ty = t;
        break;
      }
    if (ty == 0) return fail(LBF_E_UNSUPPORTED, "no tile height fits %d sites per lane", sites);
  }
  h->lane_sites = sites;
  h->tile_rows = ty;
  h->shape_set = true;
  plan(h);
  return LBF_OK;
}

int lbfast_set_adjoint_launch(lbfast_t h, int sites, int tile_rows) {
  g_err.clear();
  if (int rc = check_handle(h)) return rc;
  if (sites < 0 || sites > 3) return fail(LBF_E_ARG, "sites must be 0, 1, 2 or 3");
  if (tile_rows != 0 && tile_rows != 4 && tile_rows != 6 && tile_rows != 8 && tile_rows != 14)
    return fail(LBF_E_ARG, "tile_rows must be 0, 4, 6, 8 or 14");
  const int S = sites ? sites : 1;
  const int ty = tile_rows ? tile_rows : (h->p.storage == LBF_F64 ? 6 : 8);
  if (S > 1) {
    if (h->p.storage != LBF_F32)
      return fail(LBF_E_UNSUPPORTED, "two or three sites per lane: F32 storage only");
    if ((S == 2 && h->p.nx % 2 != 0) || (S == 3 && h->p.nx % 3 != 0))
      return fail(LBF_E_UNSUPPORTED, "nx must be divisible by the sites per lane");
    if (ty > 6 || (h->p.lattice == LBF_D3Q27 && ty != 4) ||
        (h->p.lattice == LBF_D3Q19 && ty != 4 && ty != 6))
      return fail(LBF_E_UNSUPPORTED,
                  "two or three sites per lane: 4- or 6-row tiles (D3Q27: 4 rows)");
  }
  h->adj_sites = sites;
  h->adj_rows = tile_rows;
  return LBF_OK;
}

int lbfast_step(lbfast_t h, int64_t n) {
  g_err.clear();
  if (int rc = check_handle(h)) return rc;
  if (n < 0) return fail(LBF_E_ARG, "n must be >= 0");
  if (n == 0) return LBF_OK;
  if (!h->scales_fixed) return fail(LBF_E_STATE, "16-bit scales not set: call set_moments first");
  DeviceGuard g(h->device);
  lbf::StepArgs a;
  if (int rc = step_args(h, &a)) return rc;
  for (int64_t s = 0; s < n; ++s) {
    a.src = h->buf[h->cur];
    a.dst = h->buf[h->cur ^ 1];
    a.sr_seed = step_seed(h->steps_done++);
    if (h->two_phase) {
      // phi(t+1) first: the step computes F(t+1) from it for the correction
      lbf::PhaseArgs pa = phase_args(h);
      hipError_t e = lbf::launch_phase_step(h->p.storage, pa, h->phase, h->stream);
      if (e != hipSuccess) return hip_fail(e, "phase-field launch");
      a.Ffield = h->Fph[h->pcur];
      a.Fout = h->Fph[h->pcur ^ 1];
      a.phi_dst = h->phi[h->pcur ^ 1];
      a.beta = pa.beta;
      a.kappa = pa.kappa;
      for (int k = 0; k < 3; ++k) a.Fb[k] = pa.Fb[k];
      a.contrast = pa.contrast;
      if (variable_properties(h)) a.phi_src = h->phi[h->pcur];
    }
    if (int rc = launch_forward(h, a)) return rc;
    h->cur ^= 1;
    if (h->two_phase) h->pcur ^= 1;
  }
  return LBF_OK;
}

int lbfast_set_form(lbfast_t h, int form) {
  g_err.clear();
  if (int rc = check_handle(h)) return rc;
  if (form != LBF_FORM_AUTO && form != LBF_FORM_MARCH && form != LBF_FORM_ONE_PLANE)
    return fail(LBF_E_ARG, "unknown form %d", form);
  if (form == LBF_FORM_ONE_PLANE) {
    if (is_16bit(h->p.storage))
      return fail(LBF_E_UNSUPPORTED, "16-bit storage has no one-plane form");
    if (ceil_div(h->p.nx, 64) * ceil_div(h->p.ny, lbf::kSlabRows) * h->p.nz > (1 << 20))
      return fail(LBF_E_UNSUPPORTED, "the one-plane form is for small grids");
  }
  h->form = form;
  plan(h);
  return LBF_OK;
}

int lbfast_default_launch(const lbfast_params* p, int compute_units, int force_field,
                          const lbfast_phase_params* pp, int what, lbfast_launch_info* out) {
  g_err.clear();
  if (int rc = validate(p)) return rc;
  if (!out) return fail(LBF_E_ARG, "out is NULL");
  if (force_field && pp) return fail(LBF_E_ARG, "the two-component variant has no force field");
  if (pp && pp->struct_size != sizeof(lbfast_phase_params))
    return fail(LBF_E_ARG, "phase params struct_size = %u, expected %zu", pp->struct_size,
                sizeof(lbfast_phase_params));
  if (pp && p->storage == LBF_F16SU)
    return fail(LBF_E_UNSUPPORTED, "the two-component variant does not cover LBF_F16SU storage");
  if (compute_units < 0) return fail(LBF_E_ARG, "compute_units must be >= 0");
  lbfast_ctx h;
  if (compute_units) h.cus = compute_units;
  set_params(&h, p);
  if (force_field) {
    h.Ffield = out;  // any address: only whether there is one counts here
    model_launch(&h);
    plan(&h);
  }
  if (pp) {
    h.pp = *pp;
    h.two_phase = true;
    two_phase_launch(&h);
  }
  *out = lbfast_launch_info{};
  if (what >= LBF_LAUNCH_SET_F64 && what <= LBF_LAUNCH_GET_F32) {
    out->blocks = lbf::whole_state_blocks(
        p->storage, what == LBF_LAUNCH_SET_F64 || what == LBF_LAUNCH_GET_F64 ? LBF_F64 : LBF_F32,
        what >= LBF_LAUNCH_GET_F64, h.N);
    out->block_threads = lbf::kConvertThreads;
    return LBF_OK;
  }
  if (what == LBF_LAUNCH_PHASE || what == LBF_LAUNCH_FORCE) {
    if (!pp) return fail(LBF_E_ARG, "a launch of the two-component variant");
    const lbf::PassGeom& g = what == LBF_LAUNCH_PHASE ? h.phase : h.force;
    out->lane_sites = 1;
    out->tile_rows = g.rows;
    out->z_chunk = g.zchunk;
    out->blocks = g.blocks;
    out->block_threads = 64 * g.rows;
    return LBF_OK;
  }
  Launch l = h.step;
  if (what == LBF_LAUNCH_ADJOINT) {
    if (int rc = check_adjoint_args(&h, 1, 1)) return rc;
    l = adjoint_launch(&h);
  } else if (what != LBF_LAUNCH_STEP) {
    return fail(LBF_E_ARG, "unknown launch %d", what);
  }
  out->one_plane = l.slab;
  out->lane_sites = l.lane_sites;
  out->tile_rows = l.rows;
  out->z_chunk = l.zchunk;
  out->contiguous = l.xcd_remap;
  out->plain_stores = l.slab || l.cached;
  out->blocks = static_cast<int64_t>(l.tiles_x) * l.tiles_y * l.zchunks;
  out->block_threads = 64 * (l.rows + 2);
  return LBF_OK;
}

int lbfast_enable_two_phase(lbfast_t h, const lbfast_phase_params* pp) {
  g_err.clear();
  if (int rc = check_handle(h)) return rc;
  if (!pp) return fail(LBF_E_ARG, "phase params is NULL");
  if (pp->struct_size != sizeof(lbfast_phase_params))
    return fail(LBF_E_ARG, "phase params struct_size = %u, expected %zu", pp->struct_size,
                sizeof(lbfast_phase_params));
  if (pp->reserved0 != 0) return fail(LBF_E_ARG, "reserved0 must be zero");
  if (!std::isfinite(pp->sigma) || pp->sigma < 0) return fail(LBF_E_ARG, "sigma must be >= 0");
  if (!std::isfinite(pp->width) || !(pp->width > 0)) return fail(LBF_E_ARG, "width must be > 0");
  if (!std::isfinite(pp->diffusivity) || pp->diffusivity < 0)
    return fail(LBF_E_ARG, "diffusivity must be >= 0");
  if (!std::isfinite(pp->rho_l) || !std::isfinite(pp->rho_h) || !(pp->rho_l > 0) ||
      !(pp->rho_h > 0))
    return fail(LBF_E_ARG, "phase densities must be finite and > 0");
  if (!std::isfinite(pp->tau_l) || !std::isfinite(pp->tau_h) || !(pp->tau_l > 0.5) ||
      !(pp->tau_h > 0.5))
    return fail(LBF_E_ARG, "phase relaxation times must be finite and > 1/2");
  if (h->p.bc[0] != LBF_PERIODIC || h->p.bc[2] != LBF_PERIODIC)
    return fail(LBF_E_UNSUPPORTED, "walls are supported on the y axis only");
  if (h->p.storage == LBF_F16SU)
    return fail(LBF_E_UNSUPPORTED, "the two-component variant does not cover LBF_F16SU storage");
  if (h->Ffield) return fail(LBF_E_STATE, "a per-site force field is set");
  if (h->two_phase) return fail(LBF_E_STATE, "two-component variant already enabled");
  DeviceGuard g(h->device);
  const size_t c = compute_bytes(h);
  const size_t pb = static_cast<size_t>(h->N) * c;
  hipError_t e = hipSuccess;
  void** slots[4] = {&h->phi[0], &h->phi[1], &h->Fph[0], &h->Fph[1]};
  const size_t sizes[4] = {pb, pb, 3 * pb, 3 * pb};
  for (int i = 0; i < 4 && e == hipSuccess; ++i) e = hipMalloc(slots[i], sizes[i]);
  for (int i = 0; i < 4 && e == hipSuccess; ++i)
    e = lbf::launch_zero(*slots[i], static_cast<int64_t>(sizes[i]), h->stream);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    for (int i = 0; i < 4; ++i)
      if (*slots[i]) {
        (void)hipFree(*slots[i]);
        *slots[i] = nullptr;
      }
    return fail(LBF_E_NOMEM, "two-component buffers: %s", hipGetErrorString(e));
  }
  h->pp = *pp;
  h->two_phase = true;
  h->pcur = 0;
  two_phase_launch(h);
  // F(0) of phi = 0: the body force alone
  lbf::PhaseArgs pa = phase_args(h);
  pa.phi_out = h->phi[0];
  pa.F = h->Fph[0];
  e = lbf::launch_capillary_force(h->p.storage, pa, h->force, h->stream);
  if (e != hipSuccess) return hip_fail(e, "capillary force");
  return LBF_OK;
}

int lbfast_set_phase(lbfast_t h, const void* phi, int dtype, int on_device) {
  g_err.clear();
  if (int rc = check_handle(h)) return rc;
  if (!h->two_phase) return fail(LBF_E_STATE, "two-component variant not enabled");
  if (!phi) return fail(LBF_E_ARG, "phi is NULL");
  if (dtype != LBF_F64 && dtype != LBF_F32) return fail(LBF_E_ARG, "dtype must be F64 or F32");
  if (on_device != 0 && on_device != 1) return fail(LBF_E_ARG, "on_device must be 0 or 1");
  DeviceGuard g(h->device);
  const size_t ub = (dtype == LBF_F64) ? 8 : 4;
  const size_t bytes = static_cast<size_t>(h->N) * ub;
  const void* src = phi;
  void* staging = nullptr;
  hipError_t e = hipSuccess;
  if (!on_device) {
    e = hipMalloc(&staging, bytes);
    if (e != hipSuccess) {
      (void)hipGetLastError();
      return fail(LBF_E_NOMEM, "staging allocation failed");
    }
    e = hipMemcpyAsync(staging, phi, bytes, hipMemcpyHostToDevice, h->stream);
    src = staging;
  }
  if (e == hipSuccess)
    e = lbf::launch_convert(h->p.storage, dtype, src, 0, h->phi[h->pcur], h->N, h->stream);
  if (e == hipSuccess) {
    lbf::PhaseArgs pa = phase_args(h);
    pa.phi_out = h->phi[h->pcur];
    pa.F = h->Fph[h->pcur];
    e = lbf::launch_capillary_force(h->p.storage, pa, h->force, h->stream);
  }
  if (staging) {
    hipError_t e2 = hipStreamSynchronize(h->stream);
    if (e == hipSuccess) e = e2;
    (void)hipFree(staging);
  }
  if (e != hipSuccess) return hip_fail(e, "set_phase");
  return LBF_OK;
}

int lbfast_get_phase(lbfast_t h, void* phi, int dtype, int on_device) {
  g_err.clear();
  if (int rc = check_handle(h)) return rc;
  if (!h->two_phase) return fail(LBF_E_STATE, "two-component variant not enabled");
  if (!phi) return fail(LBF_E_ARG, "phi is NULL");
  if (dtype != LBF_F64 && dtype != LBF_F32) return fail(LBF_E_ARG, "dtype must be F64 or F32");
  if (on_device != 0 && on_device != 1) return fail(LBF_E_ARG, "on_device must be 0 or 1");
  DeviceGuard g(h->device);
  const size_t ub = (dtype == LBF_F64) ? 8 : 4;
  const size_t bytes = static_cast<size_t>(h->N) * ub;
  void* dst = phi;
  void* staging = nullptr;
  hipError_t e = hipSuccess;
  if (!on_device) {
    e = hipMalloc(&staging, bytes);
    if (e != hipSuccess) {
      (void)hipGetLastError();
      return fail(LBF_E_NOMEM, "staging allocation failed");
    }
    dst = staging;
  }
  e = lbf::launch_convert(h->p.storage, dtype, h->phi[h->pcur], 1, dst, h->N, h->stream);
  if (e == hipSuccess && staging)
    e = hipMemcpyAsync(phi, staging, bytes, hipMemcpyDeviceToHost, h->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
  if (staging) (void)hipFree(staging);
  if (e != hipSuccess) return hip_fail(e, "get_phase");
  return LBF_OK;
}

int lbfast_forward_checkpointed(lbfast_t h, int64_t nsteps, int64_t every, void* ckpt_dev) {
  g_err.clear();
  if (int rc = check_handle(h)) return rc;
  if (int rc = check_adjoint_args(h, nsteps, every)) return rc;
  if (nsteps > 0 && !ckpt_dev) return fail(LBF_E_ARG, "ckpt_dev is NULL");
  if (reinterpret_cast<uintptr_t>(ckpt_dev) & 255)
    return fail(LBF_E_ARG, "ckpt_dev must be 256-byte aligned");
  DeviceGuard g(h->device);
  const size_t bytes = lbfast_buffer_bytes(&h->p);
  lbf::StepArgs a;
  if (int rc = step_args(h, &a)) return rc;
  char* ck = static_cast<char*>(ckpt_dev);
  if (every == 1 && nsteps > 0) {
    // every state is kept: each step writes straight into the next slot, and
    // only the last one (the final state, which has no slot) into the buffer
    hipError_t e = hipMemcpyAsync(ck, h->buf[h->cur], bytes, hipMemcpyDeviceToDevice, h->stream);
    if (e != hipSuccess) return hip_fail(e, "checkpoint copy");
    for (int64_t t = 0; t < nsteps; ++t) {
      a.src = ck + t * bytes;
      a.dst = (t + 1 < nsteps) ? static_cast<void*>(ck + (t + 1) * bytes) : h->buf[h->cur ^ 1];
      if (int rc = launch_forward(h, a)) return rc;
    }
    h->cur ^= 1;
    return LBF_OK;
  }
  if (nsteps == 0) return LBF_OK;
  // The initial state is copied; a later checkpoint is written into its slot by
  // the step that makes it, and read from there by the next one.  The other
  // states go to the buffers that plain steps would put them in, so that a
  // launch recorded before (a captured graph of an even number of steps) still
  // finds the current state where it was.
  hipError_t e = hipMemcpyAsync(ck, h->buf[h->cur], bytes, hipMemcpyDeviceToDevice, h->stream);
  if (e != hipSuccess) return hip_fail(e, "checkpoint copy");
  const void* at = h->buf[h->cur];
  for (int64_t t = 0; t < nsteps; ++t) {
    a.src = at;
    if ((t + 1) % every == 0 && t + 1 < nsteps)
      a.dst = ck + (t + 1) / every * bytes;
    else
      a.dst = h->buf[h->cur ^ 1];
    if (int rc = launch_forward(h, a)) return rc;
    at = a.dst;
    h->cur ^= 1;
  }
  return LBF_OK;
}

size_t lbfast_adjoint_work_bytes(lbfast_t h, int64_t every) {
  if (!h || every < 1) return 0;
  return static_cast<size_t>(every + 2) * lbfast_buffer_bytes(&h->p);
}

int lbfast_adjoint(lbfast_t h, int64_t nsteps, int64_t every, const void* ckpt_dev,
                   const void* lambda_T_dev, void* gF_dev, void* lambda0_dev, void* work_dev) {
  g_err.clear();
  if (int rc = check_handle(h)) return rc;
  if (int rc = check_adjoint_args(h, nsteps, every)) return rc;
  if (!lambda_T_dev || !gF_dev) return fail(LBF_E_ARG, "lambda_T_dev and gF_dev are required");
  if (nsteps > 0 && (!ckpt_dev || !work_dev))
    return fail(LBF_E_ARG, "ckpt_dev and work_dev are required for nsteps > 0");
  const size_t ce = (h->p.storage == LBF_F64) ? 8 : 4;
  for (const void* p : {ckpt_dev, static_cast<const void*>(work_dev)})
    if (reinterpret_cast<uintptr_t>(p) & 255)
      return fail(LBF_E_ARG, "ckpt_dev and work_dev must be 256-byte aligned");
  for (const void* p : {lambda_T_dev, static_cast<const void*>(gF_dev),
                        static_cast<const void*>(lambda0_dev)})
    if (reinterpret_cast<uintptr_t>(p) & (ce - 1))
      return fail(LBF_E_ARG, "adjoint arrays must be aligned to the compute type");
  DeviceGuard g(h->device);
  const size_t bytes = lbfast_buffer_bytes(&h->p);
  const int64_t N = h->N;
  hipError_t e = lbf::launch_zero(gF_dev, 3 * N * static_cast<int64_t>(ce), h->stream);
  if (e != hipSuccess) return hip_fail(e, "zero dJ/dF");
  if (nsteps == 0) {
    if (lambda0_dev) {
      e = hipMemcpyAsync(lambda0_dev, lambda_T_dev, bytes, hipMemcpyDeviceToDevice, h->stream);
      if (e != hipSuccess) return hip_fail(e, "adjoint copy");
    }
    return LBF_OK;
  }
  char* work = static_cast<char*>(work_dev);
  // work: recomputed states 1..every of a segment, then two adjoint buffers
  void* lam[2] = {work + every * bytes, work + (every + 1) * bytes};
  // The first adjoint step reads lambda_T and the last one writes lambda0 where
  // they lie, unless the memory is also used for something else meanwhile:
  // lambda_T has to outlast the recomputation of the last segment, and lambda0
  // is written by a step that still reads the first states and the force.
  const int64_t nseg = (nsteps + every - 1) / every;
  const size_t fbytes = 3 * static_cast<size_t>(N) * ce;
  const size_t wbytes = lbfast_adjoint_work_bytes(h, every);
  const bool lT_direct = reinterpret_cast<uintptr_t>(lambda_T_dev) % 16 == 0 &&
                         !overlap(lambda_T_dev, bytes, work, wbytes) &&
                         !overlap(lambda_T_dev, bytes, gF_dev, fbytes) &&
                         !(nsteps == 1 && overlap(lambda_T_dev, bytes, lambda0_dev, bytes));
  const bool l0_direct = lambda0_dev && reinterpret_cast<uintptr_t>(lambda0_dev) % 16 == 0 &&
                         !overlap(lambda0_dev, bytes, work, wbytes) &&
                         !overlap(lambda0_dev, bytes, ckpt_dev, nseg * bytes) &&
                         !overlap(lambda0_dev, bytes, gF_dev, fbytes) &&
                         !overlap(lambda0_dev, bytes, h->Ffield, fbytes);
  if (!lT_direct) {
    e = hipMemcpyAsync(lam[0], lambda_T_dev, bytes, hipMemcpyDeviceToDevice, h->stream);
    if (e != hipSuccess) return hip_fail(e, "adjoint copy");
  }
  const void* lam_src = lT_direct ? lambda_T_dev : lam[0];
  int cur = 0;
  lbf::StepArgs fa, aa;
  if (int rc = step_args(h, &fa)) return rc;
  aa = fa;
  aa.gF = gF_dev;
  const Launch adj = adjoint_launch(h);
  if (int rc = set_geometry(adj, &aa)) return rc;
  const bool walls_y = h->p.bc[1] == LBF_WALLS;
  for (int64_t seg = nseg - 1; seg >= 0; --seg) {
    const int64_t len = std::min(every, nsteps - seg * every);
    char* ck = static_cast<char*>(const_cast<void*>(ckpt_dev));
    // a segment's end state is the next checkpoint, except for the last
    // segment, whose end (the final state) is recomputed; with every == 1
    // only that one state is recomputed at all
    const bool end_stored = seg + 1 < nseg;
    auto state = [&](int64_t j) -> void* {  // state at t = seg*every + j
      if (j == 0) return ck + seg * bytes;
      if (j == len && end_stored) return ck + (seg + 1) * bytes;
      return work + (j - 1) * bytes;
    };
    for (int64_t j = 0; j < (end_stored ? len - 1 : len); ++j) {  // recompute the segment
      fa.src = state(j);
      fa.dst = state(j + 1);
      if (int rc = launch_forward(h, fa)) return rc;
    }
    for (int64_t j = len - 1; j >= 0; --j) {  // sweep it backwards
      aa.src = lam_src;
      aa.dst = lam[cur ^= 1];
      if (l0_direct && seg == 0 && j == 0) aa.dst = lambda0_dev;
      aa.state_old = state(j);
      aa.state_new = state(j + 1);
      e = lbf::launch_adjoint(h->p.lattice, h->p.storage, adj.rows, walls_y, aa, h->stream);
      if (e != hipSuccess) return hip_fail(e, "adjoint launch");
      lam_src = aa.dst;
    }
  }
  if (lambda0_dev && !l0_direct) {
    e = hipMemcpyAsync(lambda0_dev, lam_src, bytes, hipMemcpyDeviceToDevice, h->stream);
    if (e != hipSuccess) return hip_fail(e, "adjoint copy");
  }
  return LBF_OK;
}

int lbfast_sync(lbfast_t h) {
  g_err.clear();
  if (int rc = check_handle(h)) return rc;
  DeviceGuard g(h->device);
  hipError_t e = hipStreamSynchronize(h->stream);
  if (e != hipSuccess) return hip_fail(e, "sync");
  return LBF_OK;
}

int lbfast_reduce(lbfast_t h, double out[5]) {
  g_err.clear();
  if (int rc = check_handle(h)) return rc;
  if (!out) return fail(LBF_E_ARG, "out is NULL");
  DeviceGuard g(h->device);
  double* d_out = h->d_partials + lbf::kReduceBlocks * 5;
  hipError_t e = lbf::launch_reduce(h->p.storage, h->buf[h->cur], h->N, h->scale, h->d_partials,
                                    d_out, h->stream);
  if (e == hipSuccess)
    e = hipMemcpyAsync(out, d_out, 5 * sizeof(double), hipMemcpyDeviceToHost, h->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
  if (e != hipSuccess) return hip_fail(e, "reduce");
  for (int k = 0; k < 5; ++k)
    if (!std::isfinite(out[k])) return fail(LBF_E_NONFINITE, "non-finite sum %d in the state", k);
  return LBF_OK;
}

int lbfast_state_ptr(lbfast_t h, void** dev_ptr) {
  g_err.clear();
  if (int rc = check_handle(h)) return rc;
  if (!dev_ptr) return fail(LBF_E_ARG, "dev_ptr is NULL");
  *dev_ptr = h->buf[h->cur];
  return LBF_OK;
}

int lbfast_get_scales(lbfast_t h, float out[10]) {
  g_err.clear();
  if (int rc = check_handle(h)) return rc;
  if (!out) return fail(LBF_E_ARG, "out is NULL");
  for (int k = 0; k < 10; ++k) out[k] = h->scale[k];
  return LBF_OK;
}

}  // extern "C"
