// C ABI and host driver of the correction (declarations and contracts in ffcz.h).
//
// Per projection round the device runs, for a 3D field n0 x n1 x n2 with
// half-spectrum rows of H+1 = n2/2+1 entries:
//   y-fwd   Z -> A   C2C along axis 1
//   x-pass  A -> A   C2C along axis 0, count violations, clip Re/Im, inverse C2C
//   ctl     one block per instance: sum the counts, decide on the device
//   y-inv   A -> A   inverse C2C along axis 1
//   z-pass  A -> Z   C2R along axis 2, 1/N, clip eps, R2C
// (2D: x-pass Z -> A, ctl, z-pass A -> Z; 1D fields: the x-pass has length 1.)
// Z therefore always holds the last-axis R2C of the iterate whose check is
// running, so when that check passes the output is the C2R of Z.  Every loop
// kernel returns at entry once its instance's done-flag is set, and the control
// kernel posts each check to pinned host memory: the host enqueues a round once
// the check before it is in (drive), or, where asked to, chunks of rounds with
// one poll of the flags each.  Small 3D fields run y-inv, z-pass and the next
// round's y-fwd as one pass over planes, which also makes the check.
//
// A plan covers B instances of one shape (B = 1 for ffcz_correct): their
// spectra are stacked, so one launch of each pass serves all of them, while
// every instance keeps its own bounds, counts and done-flag.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <climits>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <mutex>
#include <map>
#include <memory>
#include <string>
#include <thread>
#include <vector>

#include "../../include/ffcz.h"
#include "common.hpp"
#include "kernels_bounds.hpp"
#include "kernels_ctl.hpp"
#include "kernels_edit.hpp"
#include "kernels_huff.hpp"
#include "kernels_plane.hpp"
#include "kernels_sig.hpp"
#include "launch.hpp"
#include "posts.hpp"
#include "sig_dispatch.hpp"

namespace ffcz {
hipError_t launch_col_f32(int mode, int L, int v, const void* args, int64_t nb, hipStream_t s);
hipError_t launch_col_f64(int mode, int L, int v, const void* args, int64_t nb, hipStream_t s);
hipError_t launch_row_f32(int mode, int H, int v, const void* args, int64_t nb, hipStream_t s);
hipError_t launch_row_f64(int mode, int H, int v, const void* args, int64_t nb, hipStream_t s);
hipError_t launch_row_f64_f32io(int mode, int H, int v, const void* args, int64_t nb, hipStream_t s);
hipError_t launch_sig_f32(int mode, int lgMc, const void* args, int nb, hipStream_t s);
hipError_t launch_sig_f64(int mode, int lgMc, const void* args, int nb, hipStream_t s);
hipError_t launch_sigt_f64(int mode, int iodt, int lgMc, const void* args, int nb, hipStream_t s);
hipError_t launch_edit_row_f32(int mode, int H, const void* args, int64_t nb, hipStream_t s);
hipError_t launch_edit_row_f64(int mode, int H, const void* args, int64_t nb, hipStream_t s);
hipError_t launch_edit_col_f32(int mode, int L, const void* args, int64_t nb, hipStream_t s);
hipError_t launch_edit_col_f64(int mode, int L, const void* args, int64_t nb, hipStream_t s);
hipError_t launch_plane_f32(int Ly, int H, const void* args, int64_t nb, hipStream_t s);
hipError_t launch_plane_f64(int Ly, int H, const void* args, int64_t nb, hipStream_t s);
hipError_t launch_bounds_row_f32(int mode, int H, int vv, const void* args, int64_t nb, hipStream_t s);
hipError_t launch_bounds_row_f64(int mode, int H, int vv, const void* args, int64_t nb, hipStream_t s);
hipError_t launch_bounds_col_f32(int mode, int L, const void* args, int64_t nb, hipStream_t s);
hipError_t launch_bounds_col_f64(int mode, int L, const void* args, int64_t nb, hipStream_t s);

// Which instantiation family runs a mode: the loop in the data type, set-up and
// verification in FP64 (SigArgs<double>).
bool sig_mode_fp64(int mode, int iodt) {
  const bool loop = mode == SIG_RUN || mode == SIG_RUNL || mode == SIGT_EPS0 || mode == SIGT_CIN || mode == SIGT_RMUL ||
                    mode == SIGT_RMULI ||
                    mode == SIGT_RCHECK || mode == SIGT_CCHECK || mode == SIGT_CSPAT || mode == SIGT_Y;
  return !loop || iodt == 1;
}

// iodt: data type of the batch; nsig: signals of the length class (the launch covers their tiles)
hipError_t launch_sig(int iodt, int mode, int lgMc, const void* args, int nsig, hipStream_t s) {
  const bool verify_t = mode == SIGT_VCOL || mode == SIGT_VROW || mode == SIGT_VCOL2;
  const bool setup = mode == SIG_SETUP || mode == SIGT_CHIRP || mode == SIGT_BCOL || mode == SIGT_BROW;
  if (iodt == 0) {
    if (verify_t) return launch_sigt_f64(mode, 0, lgMc, args, nsig, s);
    if (setup) return launch_sig_f64(mode, lgMc, args, nsig, s);
    return launch_sig_f32(mode, lgMc, args, nsig, s);
  }
  if (sig_tiled(mode) && !setup) return launch_sigt_f64(mode, 1, lgMc, args, nsig, s);
  return launch_sig_f64(mode, lgMc, args, nsig, s);
}

// Rows per row tile of the per-signal kernel (mirror of SigGeom).
int sig_rows_per_tile(int tdt, int lgMc) {
  const int MA = 1 << ((lgMc + 1) / 2), MB = (1 << lgMc) / MA;
  const int PA = MA / pick_E(MA), PB = MB / pick_E(MB);
  const int NT = imin3(sig_tile_lanes((int64_t)1 << lgMc), MA * PB, MB * PA);
  (void)tdt;
  return NT / PA;
}

int col_block_cols(int dtype, int L, int v) { return dtype == 0 ? tile_cols<float>(L, v) : tile_cols<double>(L, v); }
int row_block_rows(int dtype, int H, int v) { return dtype == 0 ? tile_rows<float>(H, v) : tile_rows<double>(H, v); }

hipError_t launch_col(int dtype, int mode, int L, int v, const void* args, int64_t nb, hipStream_t s) {
  if (mode == COL_XEDIT || mode == COL_XUNDO)  // edit bookkeeping: default tiles only
    return dtype == 0 ? launch_edit_col_f32(mode, L, args, nb, s) : launch_edit_col_f64(mode, L, args, nb, s);
  if (mode == COL_XPASSP || mode == COL_VERIFYP)  // pointwise bounds: default tiles only
    return dtype == 0 ? launch_bounds_col_f32(mode, L, args, nb, s) : launch_bounds_col_f64(mode, L, args, nb, s);
  return dtype == 0 ? launch_col_f32(mode, L, v, args, nb, s) : launch_col_f64(mode, L, v, args, nb, s);
}
}  // namespace ffcz

using namespace ffcz;

// Scratch of ffcz_correct_noalloc: a fixed device array, one copy per GPU, held until the
// process ends.
constexpr size_t kScratchBytes = (size_t)FFCZ_NOALLOC_SCRATCH_BYTES;
static __device__ __align__(256) char scratch[kScratchBytes];

namespace {

thread_local std::string g_err;

int32_t fail(int32_t code, const std::string& msg) {
  g_err = msg;
  return code;
}

#define HIPCHK(expr)                                                                  \
  do {                                                                                \
    hipError_t e_ = (expr);                                                           \
    if (e_ != hipSuccess)                                                             \
      return fail(FFCZ_E_HIP, std::string(#expr) + ": " + hipGetErrorString(e_));     \
  } while (0)

// ---------------------------------------------------------------------------
// Optional per-pass timing: HIP events recorded on the call's stream around
// every launch.  Launches that return at entry because the loop already
// finished are dropped once the call knows its round count.
enum ProfKind {
  PK_INIT = 0, PK_YFWD, PK_XPASS, PK_YINV, PK_ZPASS, PK_FINAL, PK_VZ, PK_VY, PK_VX, PK_BZ, PK_BY, PK_BX,
  PK_COUNT
};
struct ProfEv {
  hipEvent_t a, b;
  int kind, round;
  int keep;  // -1: undecided (loop launch), 0: drop, 1: keep
};
struct Profiler {
  bool on = false;
  uint32_t kinds = 0;  // kinds timed (bit per kind); 0: every kind
  std::vector<ProfEv> pending;
  std::vector<hipEvent_t> pool;
  double ms[PK_COUNT] = {0};
  int64_t cnt[PK_COUNT] = {0};
  hipEvent_t get() {
    if (!pool.empty()) {
      hipEvent_t e = pool.back();
      pool.pop_back();
      return e;
    }
    hipEvent_t e = nullptr;
    if (hipEventCreate(&e) != hipSuccess) return nullptr;
    return e;
  }
};
thread_local Profiler g_prof;

// Wrap one launch.  round < 0 marks launches that always do work.
template <typename F>
hipError_t timed(int kind, int round, hipStream_t s, F&& launch) {
  if (!g_prof.on || (g_prof.kinds != 0 && !((g_prof.kinds >> kind) & 1u))) return launch();
  ProfEv ev{g_prof.get(), g_prof.get(), kind, round, round < 0 ? 1 : -1};
  if (ev.a) (void)hipEventRecord(ev.a, s);
  hipError_t e = launch();
  if (ev.b) (void)hipEventRecord(ev.b, s);
  if (ev.a && ev.b) g_prof.pending.push_back(ev);
  return e;
}

// Decide which loop launches of the finished call did work.
void prof_settle(int rounds) {
  for (auto& ev : g_prof.pending) {
    if (ev.keep != -1) continue;
    if (ev.kind == PK_YFWD || ev.kind == PK_XPASS) ev.keep = ev.round <= rounds;
    else ev.keep = ev.round < rounds;
  }
}

constexpr int kMaxLast = 4096;  // last axis (H <= 2048)

bool is_pow2(int64_t v) { return v >= 1 && (v & (v - 1)) == 0; }

size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// squeeze unit extents
int squeeze(int32_t ndim, const int64_t* shape, int64_t* sq) {
  int nd = 0;
  for (int i = 0; i < ndim; ++i)
    if (shape[i] > 1) sq[nd++] = shape[i];
  return nd;
}

// Fields the multidimensional plan does not take -- after squeezing, a single point or
// one axis whose length is not a power of two in [2, 4096] -- run on the 1D signal path
// (four-step or Bluestein DFT of any length up to 2^19) as a batch of one.
bool route_1d(int32_t ndim, const int64_t* shape) {
  if (ndim < 1 || ndim > 3 || !shape) return false;
  for (int i = 0; i < ndim; ++i)
    if (shape[i] < 1) return false;
  int64_t sq[3];
  const int nd = squeeze(ndim, shape, sq);
  if (nd == 0) return true;
  return nd == 1 && !(is_pow2(sq[0]) && sq[0] >= 2 && sq[0] <= kMaxLast);
}

ffcz_instance one_instance(int32_t ndim, const int64_t* shape, const void* x, const void* xb, void* y, double E,
                           double D) {
  ffcz_instance in;
  memset(&in, 0, sizeof(in));
  in.ndim = ndim;
  for (int i = 0; i < 3; ++i) in.shape[i] = i < ndim ? shape[i] : 1;
  in.x_orig = x;
  in.x_base = xb;
  in.x_out = y;
  in.eps_s = E;
  in.delta_f = D;
  return in;
}

// Partial-sum slots of the on-device margin reduction of one field: a field of
// n points uses ulp_slots(n) of them (about 16 Ki points per slot), the same
// in a single call and in a batch, so both derive the same mu.
constexpr int kUlpSlots = 1024;
__host__ __device__ inline int ulp_slots(int64_t n) {
  const int64_t k = (n + 16383) / 16384;
  return (int)(k < 1 ? 1 : (k > kUlpSlots ? kUlpSlots : k));
}

struct Plan {
  int dt = 0;        // 0 f32, 1 f64
  int nd = 0;        // squeezed ndim
  int64_t B = 1;     // instances of this shape
  int64_t n[3] = {1, 1, 1};
  int64_t N = 1;     // points per instance
  int H = 0;         // n_last / 2
  int64_t ncols = 0; // H + 1
  int64_t pitch = 0; // complex entries per spectrum row (working type)
  int64_t pitch64 = 0;
  // complex entries per x-plane (3D: n1 rows plus one 128-byte line, so that the x-direction
  // passes do not stride by a round multiple of the memory interleave; else a whole instance)
  int64_t plane = 0, plane64 = 0;
  int lg_rpp = 0;    // log2 of the spectrum rows per plane
  int64_t nrows = 0; // spectrum rows per instance
  int Lx = 1, Ly = 0;
  int Ez = 1, Ey = 1, Ex = 1;
  int64_t twz = 0, twy = 0, twx = 0, twz8 = 0, twT = 0;  // twz8: last-axis tables of the radix-8 plan
  int Ez8 = 1;
  // tile variants of the loop passes (y-forward/inverse, x-pass, last-axis init/loop/final)
  int vy = 0, vx = 0, vz = 0;
  // blocks of each pass per instance (one partial slot per block)
  bool planes = false;  // the plane pass (kernels_plane.hpp) in place of y-inverse, last axis, y-forward
  int64_t zbpi = 0, ibpi = 0, vzbpi = 0, xbpi = 0, vxbpi = 0;  // ibpi: the init pass (default tiles)
  int64_t pmax = 0;
  size_t off_state = 0, off_ulp = 0, off_viol = 0, off_init = 0, off_part = 0, off_twT = 0, off_tw64 = 0, off_Z = 0,
         off_A = 0, off_W = 0, bytes = 0;
  int32_t max_iter = 0;
  int64_t s_row_w32 = 0, s_plane_bytes = 0, f_row_bytes = 0, f_plane_bytes = 0;
};

struct StateInit {
  double E, Ep, Delta, Dc, Dp, inv_n, mu, mu_s;
  int32_t max_iter, fixed, record_masks, pad;
  const void* px;
  const void* pxb;
  void* py;
  const void* pE;
  const void* pD;
  int32_t disk, pad2;
};

// Check threshold and projection bound of the f-cube.  An FP64 output is
// checked against Delta and projected onto Delta (1 - mu) (Sec. IV-B).  An FP32
// output moves every spectral component by up to mu Delta when it is rounded,
// and a coefficient accepted just below the check is never clipped, so the
// check runs mu Delta below Delta and the projection mu Delta below the check.
__host__ __device__ void spectral_thresholds(int dt, double delta, double mu, double* dc, double* dp) {
  const double rho = dt == FFCZ_F64 ? 0.0 : mu;
  *dc = delta * (1.0 - rho);
  *dp = delta * (1.0 - rho - mu);
}

int ceil_lg(int64_t v) {
  int r = 0;
  while ((int64_t(1) << r) < v) ++r;
  return r;
}

// The FP64 last-axis verification pass runs the radix-8 plan: half the registers
// per lane of radix 16, so twice the lanes of an FP64 row tile stay resident.
constexpr int kVerifyRowPlan = 2;

// FP64 fields: the closing pass runs on the radix-8 tiles of the verification and, when
// verification is on, goes on to the verification's last-axis R2C in the same pass (x and
// y read once): rows of up to 512 entries, where those tiles still hold 4 or more rows.  The
// closing pass takes the same form with verification off, so y does not depend on it.  (For
// FP32 fields the fused pass would move the closing C2R into FP64 arithmetic, and measured
// slower than the two passes.)
bool final_fused(const Plan& p) { return p.dt == FFCZ_F64 && p.H >= 2 && p.H <= 512; }

// Choose the loop passes' tile variants and the per-instance block counts that follow.
// Plan of the init, closing and adjoint last-axis passes: the direct form (variant 3)
// when the loop pass runs it on 128- or 256-entry FP32 rows, else the default tiles
// (the closing pass of FP64 fields with rows of up to 512 entries: see final_fused).
bool has_direct(const Plan& p) { return p.dt == FFCZ_F32 && (p.H == 128 || p.H == 256); }
int init_variant(const Plan& p) { return p.vz >= 3 && has_direct(p) ? p.vz : 0; }
// Last-axis plan of calls with masks (and of the adjoint) where the table holds none: nothing is
// timed for them, and a mask bit is a decision that another rounding can turn, so the direct
// form that keeps the default plan's bits (256^3 FP32, loop pass 39.9 -> 31.8 us, adjoint pass 33.1;
// a gradient of 50 rounds 12.81 -> 12.25 ms).
int masked_variant(const Plan& p, int vz) { return vz == 0 && has_direct(p) ? 4 : vz; }

// Neighbouring column tiles that read parts of the same 128-byte lines (1 when a tile row fills
// a line), and the tiles per outer index, padded to a multiple of that so that each group of
// neighbours runs on one XCD (xcd_tile; padding tiles hold no column).  FFCZ_XCD_ORDER=0 keeps
// the plain order (for measurement); both orders give identical bits.
bool xcd_order_on() {
  static const bool on = [] {
    const char* e = getenv("FFCZ_XCD_ORDER");
    return !(e && e[0] == '0');
  }();
  return on;
}
int col_line_share(int dt, int L, int v) {
  const int row_bytes = col_block_cols(dt, L, v) * (dt == FFCZ_F32 ? 8 : 16);
  return (xcd_order_on() && row_bytes < 128) ? 128 / row_bytes : 1;
}
int64_t col_tiles(int dt, int L, int v, int64_t ncols) {
  const int C = col_block_cols(dt, L, v), k = col_line_share(dt, L, v);
  return ((ncols + C - 1) / C + k - 1) / k * k;
}

void set_variants(Plan& p, int vy, int vx, int vz) {
  p.vy = vy;
  p.vx = vx;
  p.vz = vz;
  p.planes = false;
  const int64_t outer_x = p.nd == 3 ? p.n[1] : 1;
  const int Rz = row_block_rows(p.dt, p.H, vz), Rz64 = row_block_rows(1, p.H, kVerifyRowPlan);
  p.zbpi = (p.nrows + Rz - 1) / Rz;
  const int Ri = row_block_rows(p.dt, p.H, init_variant(p));
  p.ibpi = (p.nrows + Ri - 1) / Ri;
  p.vzbpi = (p.nrows + Rz64 - 1) / Rz64;
  p.xbpi = outer_x * col_tiles(p.dt, p.Lx, vx, p.ncols);
  p.vxbpi = outer_x * col_tiles(FFCZ_F64, p.Lx, 0, p.ncols);
}

int32_t make_plan(int32_t dtype, int32_t ndim, const int64_t* shape, int32_t max_iter, int64_t B, Plan& p) {
  if (dtype != FFCZ_F32 && dtype != FFCZ_F64) return fail(FFCZ_E_INVALID, "dtype must be FFCZ_F32 or FFCZ_F64");
  if (ndim < 1 || ndim > 3 || shape == nullptr) return fail(FFCZ_E_SHAPE, "ndim must be 1..3");
  if (max_iter < 0) return fail(FFCZ_E_INVALID, "max_iter must be >= 0");
  p = Plan();
  p.dt = dtype;
  p.max_iter = max_iter;
  p.B = B;
  for (int i = 0; i < ndim; ++i)
    if (shape[i] < 1) return fail(FFCZ_E_SHAPE, "every extent must be >= 1");
  int64_t sq[3];
  const int nd = squeeze(ndim, shape, sq);
  if (nd == 0) return fail(FFCZ_E_SHAPE, "a single-point field is not supported (last extent must be >= 2)");
  const int64_t maxo = dtype == FFCZ_F32 ? 2048 : 1024;
  for (int i = 0; i < nd; ++i) {
    if (!is_pow2(sq[i])) return fail(FFCZ_E_SHAPE, "extents must be powers of two");
    if (i < nd - 1 && sq[i] > maxo) return fail(FFCZ_E_SHAPE, "leading extents above the supported maximum");
  }
  const int64_t nl = sq[nd - 1];
  if (nl < 2 || nl > kMaxLast) return fail(FFCZ_E_SHAPE, "last extent must be in [2, 4096]");
  if (nd == 3 && B != 1) return fail(FFCZ_E_SHAPE, "3D instances are corrected one at a time");
  p.nd = nd;
  for (int i = 0; i < nd; ++i) p.n[i] = sq[i];
  p.N = 1;
  for (int i = 0; i < nd; ++i) p.N *= sq[i];
  p.H = (int)(nl / 2);
  p.ncols = p.H + 1;
  const int64_t cT = dtype == FFCZ_F32 ? 16 : 8;  // 128-byte pitch alignment
  p.pitch = align_up(p.ncols, cT);
  p.pitch64 = align_up(p.ncols, 8);
  p.nrows = p.N / nl;
  p.Lx = nd >= 2 ? (int)sq[0] : 1;
  p.Ly = nd == 3 ? (int)sq[1] : 0;
  p.Ez = pick_E_row(p.H);
  p.Ex = pick_E(p.Lx);
  p.Ey = p.Ly ? pick_E(p.Ly) : 1;
  p.twz = 0;
  p.twy = p.twz + host_twsize(p.H, p.Ez) + p.H;
  p.twx = p.twy + (p.Ly ? host_twsize(p.Ly, p.Ey) : 0);
  p.Ez8 = row_E(p.H, 2);
  p.twz8 = p.twx + host_twsize(p.Lx, p.Ex) + 1;
  p.twT = p.twz8 + host_twsize(p.H, p.Ez8) + p.H;
  const size_t cs = dtype == FFCZ_F32 ? 8 : 16;
  set_variants(p, 0, 0, 0);
  {
    // partial slots for the narrowest tiles any variant uses
    const int64_t outer_x = nd == 3 ? p.n[1] : 1;
    int64_t xtiles = 0;
    for (int v = 0; v < kColVariants; ++v) xtiles = std::max(xtiles, col_tiles(dtype, p.Lx, v, p.ncols));
    int Rmin = row_block_rows(dtype, p.H, 0);
    for (int v = 1; v < kRowVariants; ++v) Rmin = std::min(Rmin, row_block_rows(dtype, p.H, v));
    const int64_t zmax = (p.nrows + Rmin - 1) / Rmin, xmax = outer_x * xtiles;
    p.pmax = B * std::max(std::max(zmax, p.vzbpi), std::max(xmax, p.vxbpi));
  }
  size_t off = 0;
  p.off_state = off;
  off = align_up(off + sizeof(DevState) * (size_t)B, 256);
  p.off_ulp = off;  // margin reduction: kUlpSlots partial sums, then mu
  off = align_up(off + sizeof(double) * (kUlpSlots + 1), 256);
  p.off_viol = off;
  off = align_up(off + sizeof(unsigned long long) * ((size_t)max_iter + 2) * (size_t)B, 256);
  p.off_init = off;
  off = align_up(off + (B > 1 ? sizeof(StateInit) * (size_t)B : 0), 256);
  // partial slots: x-pass counts | z-pass counts | verify-z max | verify-x count, max
  p.off_part = off;
  off = align_up(off + sizeof(unsigned long long) * 5 * (size_t)p.pmax, 256);
  p.off_twT = off;
  off = align_up(off + cs * (size_t)p.twT, 256);
  p.off_tw64 = off;
  off = align_up(off + 16 * (size_t)p.twT, 256);
  p.off_Z = off;
  const int64_t rpp = nd == 3 ? p.n[1] : p.nrows;
  p.lg_rpp = ceil_lg(rpp);
  p.plane = rpp * p.pitch + (nd == 3 ? cT : 0);
  p.plane64 = rpp * p.pitch64 + (nd == 3 ? 8 : 0);
  const size_t nplanes = (size_t)B * (size_t)(p.nrows / rpp);
  const size_t spec = cs * nplanes * (size_t)p.plane;
  off = align_up(off + spec, 256);
  p.off_A = off;
  off = align_up(off + spec, 256);
  // the FP64 verification spectrum reuses Z..A (contiguous) once y is written; the fused
  // closing pass reads Z while it writes, so there it starts at A (free once the loop ends)
  p.off_W = final_fused(p) ? p.off_A : p.off_Z;
  const size_t spec64 = 16 * nplanes * (size_t)p.plane64;
  if (p.off_W + spec64 > off) off = align_up(p.off_W + spec64, 256);
  p.bytes = off;
  const int64_t sw64 = (nl + 63) / 64;
  const int64_t fw64 = (p.ncols + 63) / 64;
  p.s_row_w32 = 2 * sw64;
  p.s_plane_bytes = p.nrows * sw64 * 8;
  p.f_row_bytes = fw64 * 8;
  p.f_plane_bytes = p.nrows * fw64 * 8;
  return FFCZ_OK;
}

// ---------------------------------------------------------------------------
// set-up, control and statistics kernels

struct TwJob {
  int64_t off;  // complex entries from the table base
  int L, E, rtw;
};
struct TwJobs {
  TwJob j[4];
  int n;
  int dbl;  // 1: double table
};

// Stage twiddles exp(-2 pi i m r / (Ns R)) and R2C twiddles exp(-2 pi i k / 2L),
// evaluated in FP64 with an exactly reduced argument and rounded once.
__device__ __forceinline__ void write_twiddle(void* base, const TwJobs& jobs, int64_t gid) {
  int64_t acc = 0;
  for (int jj = 0; jj < jobs.n; ++jj) {
    const TwJob& jb = jobs.j[jj];
    // the stage plan of host_twsize, walked without a table (no per-lane scratch)
    const int64_t tsz = jb.E > 1 && jb.L > 1 ? host_twsize(jb.L, jb.E) : 0;
    const int64_t cnt = tsz + (jb.rtw ? jb.L : 0);
    if (gid < acc + cnt) {
      const int64_t e = gid - acc;
      double num, den;  // angle = -2 pi num / den
      if (e < tsz) {
        const int lgE = ilog2c(jb.E), a = ilog2c(jb.L) / lgE;
        const int r0 = jb.L >> (a * lgE);
        int64_t ns = r0 > 1 ? r0 : 1, off = 0;
        for (int t = 0; t < a; ++t, ns *= jb.E) {
          if (ns == 1) continue;
          const int64_t own = ns * (jb.E - 1);
          if (e < off + own) break;
          off += own;
        }
        const int64_t loc = e - off;
        const int64_t m = loc / (jb.E - 1);
        const int64_t r = loc % (jb.E - 1) + 1;
        num = (double)(m * r);
        den = (double)ns * jb.E;
      } else {
        num = (double)(e - tsz);
        den = 2.0 * jb.L;
      }
      double sn, cs;
      sincospi(-2.0 * num / den, &sn, &cs);
      if (jobs.dbl) {
        cx<double>* t = (cx<double>*)base + jb.off + e;
        *t = cx<double>{cs, sn};
      } else {
        cx<float>* t = (cx<float>*)base + jb.off + e;
        *t = cx<float>{__double2float_rn(cs), __double2float_rn(sn)};
      }
      return;
    }
    acc += cnt;
  }
}

// Lane t of nthr: the state of instance t, and its share of the words to clear.
__device__ __forceinline__ void state_init(DevState* st, int64_t B, const StateInit* arr, const StateInit& one,
                                           unsigned long long* viol, int64_t nviol, int64_t t, int64_t nthr) {
  if (t < B) {
    const StateInit p = arr ? arr[t] : one;
    DevState s;
    memset(&s, 0, sizeof(s));
    s.E = p.E;
    s.Ep = p.Ep;
    s.Delta = p.Delta;
    s.Dc = p.Dc;
    s.Dp = p.Dp;
    s.inv_n = p.inv_n;
    s.mu = p.mu;
    s.mu_s = p.mu_s;
    s.max_iter = p.max_iter;
    s.fixed = p.fixed;
    s.record_masks = p.record_masks;
    s.px = p.px;
    s.pxb = p.pxb;
    s.py = p.py;
    s.pE = p.pE;
    s.pD = p.pD;
    s.disk = p.disk;
    s.fe = 1.0 - p.mu;
    s.fc = 1.0;
    s.fp = 1.0 - p.mu;
    st[t] = s;
  }
  for (int64_t i = t; i < nviol; i += nthr) viol[i] = 0ull;
}

// Suggested FP32 margin for a field of N points with bound Delta:
// mu = max(2^-16, 8 sigma sqrt(N/2) / Delta), sigma^2 = mean(ulp(x)^2) / 12, at
// most 1/2.  Rounding y to FP32 moves each Re/Im component of its spectrum by
// sigma sqrt(N/2) rms (N independent roundings of variance ulp^2/12, half of
// each in the real part).  A non-finite sum gives 2^-16 (NaN) or 1/2 (Inf);
// such inputs stop the correction anyway.
__host__ __device__ double margin_from_ulp2(double ulp2_sum, int64_t N, double D) {
  const double sigma = sqrt(ulp2_sum / (double)N / 12.0);
  const double m = D > 0 ? 8.0 * sigma * sqrt((double)N / 2.0) / D : 0.5;
  const double lo = 0x1p-16;
  const double a = lo < m ? m : lo;
  return a < 0.5 ? a : 0.5;
}

// One field of a margin computation: x (FP32, N points) and its bound Delta.
struct MarginJob {
  const float* x;
  int64_t n;
  double D;
  int64_t sig;  // 1 + the field's position among the 1D members of a batch (0: not one)
};

// ulp(v)^2 = (nextafter(|v|, +Inf) - |v|)^2 from the exponent field e of v:
// 2^(2 max(e, 1) - 300), exact in FP64; FLT_MAX steps to Inf, Inf and NaN give NaN.
__device__ inline double ulp2f(float v) {
  const uint32_t b = __float_as_uint(v) & 0x7fffffffu;
  const uint32_t e = b >> 23;
  if (e == 255u) return __longlong_as_double(0x7ff8000000000000ll);
  if (b == 0x7f7fffffu) return __longlong_as_double(0x7ff0000000000000ll);
  const int64_t ex = 2 * (int64_t)(e > 0u ? e : 1u) - 300 + 1023;
  return __longlong_as_double(ex << 52);
}

// Partial sums of ulp(x)^2 of one field: its points are cut into nb = ulp_slots(n)
// contiguous slices of a multiple of 4 points, and block b < nb (256 lanes) stores the sum
// over slice b in part[b] (blocks past nb have nothing to do).  No
// atomics: margin_kernel adds the slots in a fixed order, so mu does not
// depend on scheduling.  Aligned slices stream 16-byte vectors, four in flight
// per lane.
__device__ __forceinline__ void ulp_part(const MarginJob& jb, int64_t b, double* part) {
  __shared__ double red[4];
  const int64_t nb = ulp_slots(jb.n);
  if (b >= nb) return;
  const int64_t slice = ((jb.n + nb - 1) / nb + 3) & ~int64_t(3);
  const int64_t lo = std::min<int64_t>(jb.n, b * slice);
  const int64_t hi = std::min<int64_t>(jb.n, lo + slice);
  const float* x = jb.x;
  double s = 0.0;
  int64_t i0 = lo;
  if (((uintptr_t)(x + lo) & 15) == 0) {
    const float4* x4 = (const float4*)(x + lo);
    const int64_t n4 = (hi - lo) >> 2;
    constexpr int U = 4;
    int64_t k = threadIdx.x;
    for (; k + (U - 1) * 256 < n4; k += U * 256) {
      float4 v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] = x4[k + u * 256];
#pragma unroll
      for (int u = 0; u < U; ++u) s += ulp2f(v[u].x) + ulp2f(v[u].y) + ulp2f(v[u].z) + ulp2f(v[u].w);
    }
    for (; k < n4; k += 256) {
      const float4 v = x4[k];
      s += ulp2f(v.x) + ulp2f(v.y) + ulp2f(v.z) + ulp2f(v.w);
    }
    i0 = lo + 4 * n4;
  }
  for (int64_t i = i0 + threadIdx.x; i < hi; i += 256) s += ulp2f(x[i]);
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) part[b] = (red[0] + red[1]) + (red[2] + red[3]);
}
// One field (jobs null) or field blockIdx.y of several, its slots from part[y * kUlpSlots] on.
__global__ void __launch_bounds__(256) ulp_part_kernel(MarginJob one, const MarginJob* jobs, double* part) {
  ulp_part(jobs ? jobs[blockIdx.y] : one, blockIdx.x, part + (int64_t)blockIdx.y * kUlpSlots);
}

// Everything a call writes or sums before its first pass, side by side in one launch: instance
// states (nbs blocks; they also clear nzero words), the twiddle tables of both precisions (nbt
// blocks each) and, where the margin comes from x, the ulp partials of x (the rest).  Three
// launches of 4-7 us in a row before: 64^3 FP64 156 -> 149 us a correction (the best of each; 150-160
// over processes), 64 x 256 x 128 FP32 230 -> 216, 2048^2 FP32 359 -> 348.
struct SetupArgs {
  DevState* st;
  int64_t B;
  const StateInit* arr;
  StateInit one;
  unsigned long long* zero;
  int64_t nzero;
  void* tw[2];
  TwJobs jobs[2];
  MarginJob ulp;
  double* part;
  int nbs, nbt;
};
__global__ void __launch_bounds__(256) setup_kernel(SetupArgs a) {
  int b = blockIdx.x;
  if (b < a.nbs) {
    state_init(a.st, a.B, a.arr, a.one, a.zero, a.nzero, (int64_t)b * 256 + threadIdx.x, (int64_t)a.nbs * 256);
    return;
  }
  b -= a.nbs;
  if (b < 2 * a.nbt) {
    const int k = b < a.nbt ? 0 : 1;
    write_twiddle(a.tw[k], a.jobs[k], (int64_t)(b - k * a.nbt) * 256 + threadIdx.x);
    return;
  }
  ulp_part(a.ulp, b - 2 * a.nbt, a.part);
}

// One block per field: add its ulp_slots(n) partial sums in a fixed order and
// derive mu.  mu_out[field] receives it when given; st (one state per field), when
// given, receives mu and the bounds that depend on it (E (1 - mu) and the
// spectral check and projection thresholds), the same values the host fills
// in when mu is supplied; so does the descriptor in sigs of a 1D member of a batch.
__global__ void __launch_bounds__(256) margin_kernel(const double* part, MarginJob one, const MarginJob* jobs, int dt,
                                                     double* mu_out, DevState* st, SigDesc* sigs = nullptr) {
  __shared__ double red[4];
  const MarginJob jb = jobs ? jobs[blockIdx.x] : one;
  const int nslot = ulp_slots(jb.n);
  const double* pp = part + (int64_t)blockIdx.x * kUlpSlots;
  double s = 0.0;
  for (int k = threadIdx.x; k < nslot; k += 256) s += pp[k];
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x != 0) return;
  const double mu = margin_from_ulp2((red[0] + red[1]) + (red[2] + red[3]), jb.n, jb.D);
  if (mu_out) mu_out[blockIdx.x] = mu;
  if (st) {
    DevState* t = st + blockIdx.x;
    t->mu = mu;
    t->Ep = t->E * (1.0 - mu);
    double dc, dp;
    spectral_thresholds(dt, t->Delta, mu, &dc, &dp);
    t->Dc = dc;
    t->Dp = dp;
  }
  if (sigs && jb.sig > 0) {  // a 1D member of a batch: its descriptor's thresholds
    SigDesc* d = sigs + (jb.sig - 1);
    d->Ep = d->E * (1.0 - mu);
    double dc, dp;
    spectral_thresholds(dt, d->Delta, mu, &dc, &dp);
    d->Dc = dc;
    d->Dp = dp;
  }
}


// max |x| partials of a field (one per slice, slices as in ulp_part_kernel), as the bits of
// a non-negative double (which order as integers).  16-byte loads, four in flight (256^3 FP32
// 20 -> 12 us).
template <typename TIO>
__global__ void __launch_bounds__(256) absmax_part_kernel(const TIO* x, int64_t n, unsigned long long* part) {
  __shared__ double red[4];
  const int64_t nb = ulp_slots(n);
  if ((int64_t)blockIdx.x >= nb) return;
  const int64_t slice = ((n + nb - 1) / nb + 3) & ~int64_t(3);
  const int64_t lo = std::min<int64_t>(n, (int64_t)blockIdx.x * slice);
  const int64_t hi = std::min<int64_t>(n, lo + slice);
  TIO mt = TIO(0);
  int64_t i0 = lo;
  constexpr int V = 16 / (int)sizeof(TIO), U = 4;
  struct alignas(16) Vec {
    TIO e[V];
  };
  if (((uintptr_t)(x + lo) & 15) == 0) {
    const Vec* xv = (const Vec*)(x + lo);
    const int64_t nv = (hi - lo) / V;
    int64_t k = threadIdx.x;
    for (; k + (U - 1) * 256 < nv; k += U * 256) {
      Vec v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] = xv[k + u * 256];
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int q = 0; q < V; ++q) mt = fmax(mt, fabs(v[u].e[q]));
    }
    for (; k < nv; k += 256) {
      const Vec v = xv[k];
#pragma unroll
      for (int q = 0; q < V; ++q) mt = fmax(mt, fabs(v.e[q]));
    }
    i0 = lo + V * nv;
  }
  for (int64_t i = i0 + threadIdx.x; i < hi; i += 256) mt = fmax(mt, fabs(x[i]));
  double m = (double)mt;
  for (int off = 32; off > 0; off >>= 1) m = fmax(m, __shfl_xor(m, off, 64));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0)
    part[blockIdx.x] = (unsigned long long)__double_as_longlong(fmax(fmax(red[0], red[1]), fmax(red[2], red[3])));
}

// Spacing of the dtype's grid just above v >= 0 (what an output of that size is rounded to).
__device__ inline double grid_spacing(int dt, double v) {
  if (dt == FFCZ_F32) {
    const float f = __double2float_rn(v);
    return (double)nextafterf(f, __builtin_huge_valf()) - (double)f;
  }
  return nextafter(v, __builtin_huge_val()) - v;
}

// Shrinks of the encoder, one block.  The paper shrinks both cubes by 2^-m so that the
// quantised edits still land inside (Sec. IV-B).  That counts each edit's own rounding
// only: the quantisation error of one domain also reaches the other through the
// transform, and the decoder rounds its output without a clamp (it does not know x).  So
// with q = safety 2^-m:
//   mu_f = max(q, mu_out)  (mu_out: the output-rounding margin of the plain correction,
//                           from the ulp partials for FP32 fields, 2^-16 for FP64),
//   mu_s = q + spacing(max|x| + E) / E  (a whole output ulp, twice its rounding error),
// capped at 1/4 and 1/2; the check runs at Delta (1 - mu_f), the f-projection at
// Delta (1 - 2 mu_f) and the s-projection at E (1 - mu_s).
__global__ void __launch_bounds__(256) encode_margin_kernel(const double* ulp_part, const unsigned long long* amax,
                                                            int64_t n, int dt, double q, DevState* st) {
  __shared__ double red[4];
  __shared__ unsigned long long redm[4];
  const int nslot = ulp_slots(n);
  double s = 0.0;
  unsigned long long mb = 0;
  for (int k = threadIdx.x; k < nslot; k += 256) {
    if (dt == FFCZ_F32) s += ulp_part[k];
    mb = mb > amax[k] ? mb : amax[k];
  }
  for (int off = 32; off > 0; off >>= 1) {
    s += __shfl_xor(s, off, 64);
    const unsigned long long o = __shfl_xor(mb, off, 64);
    mb = mb > o ? mb : o;
  }
  if ((threadIdx.x & 63) == 0) {
    red[threadIdx.x >> 6] = s;
    redm[threadIdx.x >> 6] = mb;
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  for (int w = 1; w < 4; ++w) redm[0] = redm[0] > redm[w] ? redm[0] : redm[w];
  const double xm = __longlong_as_double((long long)redm[0]);
  const double mu_out = dt == FFCZ_F32 ? margin_from_ulp2((red[0] + red[1]) + (red[2] + red[3]), n, st->Delta)
                                       : 0x1p-16;
  const double E = st->E;
  const double mu_f = fmin(fmax(mu_out, q), 0.25);
  const double mu_s = fmin(q + (E > 0.0 ? grid_spacing(dt, xm + E) / E : 0.0), 0.5);
  st->mu = mu_f;
  st->mu_s = mu_s;
  st->Ep = E * (1.0 - mu_s);
  st->Dc = st->Delta * (1.0 - mu_f);
  st->Dp = st->Delta * (1.0 - 2.0 * mu_f);
}

// Margin and threshold factors for pointwise bounds, one block.  FP64 output: mu = 2^-16 (or
// the caller's), check at D_k, project onto D_k (1 - mu) and E_n (1 - mu).  FP32 output: the
// FP32 rule of margin_kernel with Delta = the smallest spectral bound (times sqrt 2 for the
// disk, whose modulus takes the rounding noise of both parts), check at D_k (1 - mu), project
// onto D_k (1 - 2 mu).
__global__ void __launch_bounds__(256) bounds_margin_kernel(const double* ulp_part, const unsigned long long* minpart,
                                                            int nmin, int64_t n, int dt, int disk, double mu_given,
                                                            DevState* st) {
  __shared__ double red[4];
  __shared__ unsigned long long redm[4];
  const int nslot = ulp_slots(n);
  double s = 0.0;
  unsigned long long mb = ~0ull;
  if (dt == FFCZ_F32)
    for (int k = threadIdx.x; k < nslot; k += 256) s += ulp_part[k];
  for (int k = threadIdx.x; k < nmin; k += 256) mb = mb < minpart[k] ? mb : minpart[k];
  for (int off = 32; off > 0; off >>= 1) {
    s += __shfl_xor(s, off, 64);
    const unsigned long long o = __shfl_xor(mb, off, 64);
    mb = mb < o ? mb : o;
  }
  if ((threadIdx.x & 63) == 0) {
    red[threadIdx.x >> 6] = s;
    redm[threadIdx.x >> 6] = mb;
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  for (int w = 1; w < 4; ++w) redm[0] = redm[0] < redm[w] ? redm[0] : redm[w];
  double mu = mu_given;
  if (!(mu > 0.0)) {
    if (dt == FFCZ_F64) {
      mu = 0x1p-16;
    } else {
      const double dmin = redm[0] == ~0ull ? 0.0 : __longlong_as_double((long long)redm[0]);
      const double sigma = sqrt(((red[0] + red[1]) + (red[2] + red[3])) / (double)n / 12.0);
      double m = dmin > 0.0 ? 8.0 * sigma * sqrt((double)n / 2.0) / dmin : 0.5;
      if (disk && dmin > 0.0) m *= sqrt(2.0);
      mu = fmin(0.5, fmax(0x1p-16, m));
    }
  }
  const double rho = dt == FFCZ_F64 ? 0.0 : mu;
  st->mu = mu;
  st->fe = 1.0 - mu;
  st->fc = 1.0 - rho;
  st->fp = 1.0 - rho - mu;
  st->Ep = st->E * (1.0 - mu);
}

// Partials p[0..n) read by the nt lanes of a block, U independent loads in flight per lane
// (a plain strided loop waits for each load in turn: with thousands of partials that was
// most of a control kernel's time).  fold is a sum or a max of non-negative values.
template <int U, typename F>
__device__ __forceinline__ unsigned long long fold_strided(const unsigned long long* p, int64_t n, int t, int nt,
                                                           unsigned long long acc, F fold) {
  for (int64_t i0 = t; i0 < n; i0 += (int64_t)U * nt) {
    unsigned long long v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t i = i0 + (int64_t)u * nt;
      v[u] = i < n ? p[i] : 0ull;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) acc = fold(acc, v[u]);
  }
  return acc;
}
__device__ __forceinline__ unsigned long long add_u64(unsigned long long a, unsigned long long b) { return a + b; }
__device__ __forceinline__ unsigned long long max_u64(unsigned long long a, unsigned long long b) { return a > b ? a : b; }

// Per-round control, one block per instance: sum the x-pass partials into
// v_k, fold the spatial-clip partials of the z-pass that produced the checked
// iterate into the totals, and decide on the device whether the loop stops
// (Alg. 1: stop when no coefficient violates; also at the round cap, or on
// non-finite input).
__global__ void __launch_bounds__(1024) ctl_kernel(DevState* st0, unsigned long long* viol0, int64_t vstride,
                                                   const unsigned long long* xpart, int64_t xbpi,
                                                   const unsigned long long* zpart, int64_t zbpi,
                                                   int64_t ibpi, Post post) {
  __shared__ unsigned long long rx[16], rz[16];
  const int64_t b = blockIdx.x;
  DevState* st = st0 + b;
  if (*(volatile int32_t*)&st->done) return;
  const int t = threadIdx.x;
  // the checked iterate came from the init pass (round 0) or from a z-pass, whose tiles may differ
  const int64_t nz = st->round == 0 ? ibpi : zbpi;
  unsigned long long sx = fold_strided<8>(xpart + b * xbpi, xbpi, t, (int)blockDim.x, 0ull, add_u64);
  unsigned long long sz = fold_strided<8>(zpart + b * nz, nz, t, (int)blockDim.x, 0ull, add_u64);
  sx = wave_sum_u64(sx);
  sz = wave_sum_u64(sz);
  if ((t & 63) == 0) {
    rx[t >> 6] = sx;
    rz[t >> 6] = sz;
  }
  __syncthreads();
  if (t == 0) {
    unsigned long long vx = 0, vz = 0;
    for (int w = 0; w < (int)(blockDim.x + 63) / 64; ++w) {
      vx += rx[w];
      vz += rz[w];
    }
    const int k = st->round;
    record_check(st, k, vx, vz, check_stops(st, k, vx), viol0 + b * vstride, post, b);
  }
}

// Reduce the verification partials of each instance: max |y - x|,
// max(|Re|,|Im|) and the count above Delta.
__global__ void __launch_bounds__(1024) stats_kernel(DevState* st0, const unsigned long long* vz, int64_t vzbpi,
                                                     const unsigned long long* vxc, const unsigned long long* vxm,
                                                     int64_t vxbpi) {
  __shared__ unsigned long long ra[16], rb[16], rc[16];
  const int64_t inst = blockIdx.x;
  const int t = threadIdx.x;
  // max bits of non-negative doubles order as integers
  unsigned long long a = fold_strided<8>(vz + inst * vzbpi, vzbpi, t, (int)blockDim.x, 0ull, max_u64);
  unsigned long long b = fold_strided<8>(vxm + inst * vxbpi, vxbpi, t, (int)blockDim.x, 0ull, max_u64);
  unsigned long long c = fold_strided<8>(vxc + inst * vxbpi, vxbpi, t, (int)blockDim.x, 0ull, add_u64);
  for (int off = 32; off > 0; off >>= 1) {
    const unsigned long long oa = __shfl_xor(a, off, 64), ob = __shfl_xor(b, off, 64);
    a = a > oa ? a : oa;
    b = b > ob ? b : ob;
    c += __shfl_xor(c, off, 64);
  }
  if ((t & 63) == 0) {
    ra[t >> 6] = a;
    rb[t >> 6] = b;
    rc[t >> 6] = c;
  }
  __syncthreads();
  if (t == 0) {
    unsigned long long A = 0, Bm = 0, Cc = 0;
    for (int w = 0; w < (int)(blockDim.x + 63) / 64; ++w) {
      A = A > ra[w] ? A : ra[w];
      Bm = Bm > rb[w] ? Bm : rb[w];
      Cc += rc[w];
    }
    st0[inst].max_spatial_bits = A;
    st0[inst].max_spectral_bits = Bm;
    st0[inst].spectral_viol = Cc;
  }
}

// ---------------------------------------------------------------------------

struct Ctx {
  const Plan* p;
  char* ws;
  hipStream_t s;
  // edit accumulators (encoder only): spatial, one value per point; frequency, laid out as Z
  void* sacc = nullptr;
  void* facc = nullptr;
  // pointwise bounds: the (Re, Im) bound pairs laid out as Z (null: the scalar bounds)
  const void* pD = nullptr;
  Post post{nullptr, 0};  // where the control kernel tells the host of a check
  DevState* st() const { return (DevState*)(ws + p->off_state); }
  unsigned long long* viol() const { return (unsigned long long*)(ws + p->off_viol); }
  void* twT() const { return ws + p->off_twT; }
  void* tw64() const { return ws + p->off_tw64; }
  void* Z() const { return ws + p->off_Z; }
  void* A() const { return ws + p->off_A; }
  void* W() const { return ws + p->off_W; }
  unsigned long long* part(int i) const { return (unsigned long long*)(ws + p->off_part) + (size_t)i * p->pmax; }
  static constexpr int PX = 0, PZ = 1, PVZ = 2, PVX = 3;  // PVX spans two regions (count, max)
};

hipError_t launch_ctl(const Ctx& c, unsigned long long* viol, int64_t vstride) {
  hipLaunchKernelGGL(ctl_kernel, dim3((unsigned)c.p->B), dim3(1024), 0, c.s, c.st(), viol, vstride, c.part(Ctx::PX),
                     c.p->xbpi, c.part(Ctx::PZ), c.p->zbpi, c.p->ibpi, c.post);
  return hipGetLastError();
}

// States (arr, or `one`), cleared words, twiddle tables and, given x, its ulp partials.
hipError_t run_setup(const Ctx& c, const StateInit* arr, const StateInit& one, unsigned long long* zero, int64_t nzero,
                     const MarginJob* ulp = nullptr) {
  const Plan& p = *c.p;
  SetupArgs a;
  memset(&a, 0, sizeof(a));
  a.st = c.st();
  a.B = p.B;
  a.arr = arr;
  a.one = one;
  a.zero = zero;
  a.nzero = nzero;
  // table 0: working precision (read by the loop kernels); table 1: FP64 (verification)
  TwJobs* const jobs = a.jobs;
  for (int tab = 0; tab < 2; ++tab) {
    memset(&jobs[tab], 0, sizeof(TwJobs));
    jobs[tab].dbl = (tab == 1 || p.dt == FFCZ_F64) ? 1 : 0;
    int n = 0;
    jobs[tab].j[n++] = TwJob{p.twz, p.H, p.Ez, 1};
    jobs[tab].j[n++] = TwJob{p.twz8, p.H, p.Ez8, 1};
    if (p.Ly) jobs[tab].j[n++] = TwJob{p.twy, p.Ly, p.Ey, 0};
    jobs[tab].j[n++] = TwJob{p.twx, p.Lx, p.Ex, 0};
    jobs[tab].n = n;
  }
  a.tw[0] = c.twT();
  a.tw[1] = c.tw64();
  a.nbs = (int)std::min<int64_t>(1024, std::max<int64_t>(1, (std::max(p.B, nzero) + 255) / 256));
  a.nbs = (int)std::max<int64_t>(a.nbs, (p.B + 255) / 256);
  a.nbt = (int)((p.twT + 255) / 256);
  int nu = 0;
  if (ulp) {
    a.ulp = *ulp;
    a.part = (double*)(c.ws + p.off_ulp);
    nu = ulp_slots(ulp->n);
  }
  hipLaunchKernelGGL(setup_kernel, dim3((unsigned)(a.nbs + 2 * a.nbt + nu)), dim3(256), 0, c.s, a);
  return hipGetLastError();
}

// Geometry of a strided-axis pass.
struct ColGeom {
  int L;
  int64_t outer, so, s;
  int64_t mrow_i, mrow_o;
  int64_t outer_per_inst;
  int64_t pitch;  // complex entries per row of the buffer (the padded row)
};

// pitch / plane: complex entries per spectrum row / per x-plane of the buffer addressed
ColGeom geom_y(const Plan& p, int64_t pitch, int64_t plane) {  // 3D only (B = 1)
  return ColGeom{p.Ly, p.n[0], plane, pitch, 0, 0, p.n[0], pitch};
}
ColGeom geom_x(const Plan& p, int64_t pitch, int64_t plane) {
  if (p.nd == 3) return ColGeom{p.Lx, p.n[1], pitch, plane, p.n[1], 1, p.n[1], pitch};
  // 2D (and 1D, Lx = 1): one outer index per instance (a whole instance is one plane)
  return ColGeom{p.Lx, p.B, plane, pitch, 1, 0, 1, pitch};
}

template <typename T>
hipError_t run_col(int dt, int mode, int v, const ColGeom& g, const Plan& p, const void* src, void* dst,
                   const void* tw, DevState* st, unsigned long long* part, uint8_t* fmask,
                   hipStream_t s, void* fedit = nullptr, const void* bnd = nullptr, int64_t bnd_so = 0,
                   int64_t bnd_s = 0, int bnd_dbl = 0) {
  ColArgs<T> a;
  memset(&a, 0, sizeof(a));
  a.src = (const cx<T>*)src;
  a.dst = (cx<T>*)dst;
  a.so = g.so;
  a.s = g.s;
  a.ncols = (int32_t)p.ncols;
  a.ncols_pad = (int32_t)g.pitch;
  a.ncb = (int32_t)col_tiles(dt, g.L, v, p.ncols);
  a.xcd_k = col_line_share(dt, g.L, v);
  a.outer_per_inst = g.outer_per_inst;
  a.tw = (const cx<T>*)tw;
  a.st = st;
  a.part = part;
  a.part_stride = p.pmax;
  a.fmask = fmask;
  a.f_plane = p.f_plane_bytes;
  a.f_row_bytes = p.f_row_bytes;
  a.mrow_i = g.mrow_i;
  a.mrow_o = g.mrow_o;
  a.fedit = (cx<T>*)fedit;
  a.bnd = bnd;
  a.bnd_so = bnd_so;
  a.bnd_s = bnd_s;
  a.bnd_dbl = bnd_dbl;
  const int64_t nb = g.outer * a.ncb;
  return launch_col(dt, mode, g.L, v, &a, nb, s);
}

template <typename T, typename TIO>
hipError_t run_row(int tdt, int iodt, int mode, int v, const Plan& p, int64_t pitch, int64_t plane, const void* src,
                   void* dst, const void* tw, DevState* st, unsigned long long* part, uint32_t* smask,
                   hipStream_t s, int64_t spitch = -1, int64_t splane = -1, void* sedit = nullptr) {
  RowArgs<T, TIO> a;
  memset(&a, 0, sizeof(a));
  a.src = (const cx<T>*)src;
  a.dst = (cx<T>*)dst;
  a.pitch = pitch;
  a.spitch = spitch < 0 ? pitch : spitch;
  a.splane = splane < 0 ? plane : splane;
  a.rows_per_inst = p.nrows;
  const int R = row_block_rows(tdt, p.H, v);
  a.bpi = (p.nrows + R - 1) / R;
  a.tw = (const cx<T>*)tw;
  a.st = st;
  a.part = part;
  a.smask = smask;
  a.s_plane = p.s_plane_bytes / 4;
  a.s_row_w32 = (int32_t)p.s_row_w32;
  const int64_t nb = a.bpi * p.B;
  a.plane = plane;
  a.lg_rpp = p.lg_rpp;
  a.sedit = (T*)sedit;
  if (mode == ROW_INITE || mode == ROW_LOOPE || mode == ROW_DECODE)  // default tiles only
    return tdt == 0 ? launch_edit_row_f32(mode, p.H, &a, nb, s) : launch_edit_row_f64(mode, p.H, &a, nb, s);
  if (mode >= ROW_INITP && mode <= ROW_VERIFYP)  // pointwise bounds, by the field's dtype
    return iodt == 0 ? launch_bounds_row_f32(mode, p.H, v, &a, nb, s) : launch_bounds_row_f64(mode, p.H, v, &a, nb, s);
  if (tdt == 1 && iodt == 0) return launch_row_f64_f32io(mode, p.H, v, &a, nb, s);
  return tdt == 0 ? launch_row_f32(mode, p.H, v, &a, nb, s) : launch_row_f64(mode, p.H, v, &a, nb, s);
}

template <typename T>
hipError_t row_T(int mode, const Ctx& c, const void* src, void* dst, uint32_t* smask) {
  const Plan& p = *c.p;
  if (c.pD && (mode == ROW_INIT || mode == ROW_LOOP)) {
    // pointwise bounds: the staged pass on the default tiles
    return run_row<T, T>(p.dt, p.dt, mode == ROW_INIT ? ROW_INITP : ROW_LOOPP, 0, p, p.pitch, p.plane, src, dst,
                         (const char*)c.twT() + sizeof(cx<T>) * p.twz, c.st(), c.part(Ctx::PZ), smask, c.s);
  }
  if (c.sacc && (mode == ROW_INIT || mode == ROW_LOOP)) {
    // with edit bookkeeping: the staged pass on the default tiles
    return run_row<T, T>(p.dt, p.dt, mode == ROW_INIT ? ROW_INITE : ROW_LOOPE, 0, p, p.pitch, p.plane, src, dst,
                         (const char*)c.twT() + sizeof(cx<T>) * p.twz, c.st(), c.part(Ctx::PZ), smask, c.s, -1, -1,
                         c.sacc);
  }
  const int v = mode == ROW_LOOP ? p.vz : init_variant(p);
  const void* tw = (const char*)c.twT() + sizeof(cx<T>) * (v == 2 ? p.twz8 : p.twz);
  return run_row<T, T>(p.dt, p.dt, mode, v, p, p.pitch, p.plane, src, dst, tw, c.st(), c.part(Ctx::PZ), smask, c.s);
}

// The loop's x-pass: plain, with edit bookkeeping, or against pointwise bounds (the bound
// pairs share the spectrum's layout).
template <typename T>
hipError_t xpass_T(const Ctx& c, const void* src, void* dst, const void* twx, unsigned long long* px, uint8_t* fmask) {
  const Plan& p = *c.p;
  const ColGeom g = geom_x(p, p.pitch, p.plane);
  if (c.pD)
    return run_col<T>(p.dt, COL_XPASSP, 0, g, p, src, dst, twx, c.st(), px, nullptr, c.s, nullptr, c.pD, g.so, g.s,
                      p.dt == FFCZ_F64 ? 1 : 0);
  return run_col<T>(p.dt, c.facc ? COL_XEDIT : COL_XPASS, c.facc ? 0 : p.vx, g, p, src, dst, twx, c.st(), px, fmask,
                    c.s, c.facc);
}

// y-inverse, last axis and y-forward of a round in one pass over planes held in LDS.
template <typename T>
hipError_t run_planes(const Ctx& c, int r, unsigned long long* viol, int64_t vstride) {
  const Plan& p = *c.p;
  const cx<T>* twb = (const cx<T>*)c.twT();
  PlaneArgs<T> a;
  memset(&a, 0, sizeof(a));
  a.A = (cx<T>*)c.A();
  a.Z = (cx<T>*)c.Z();
  a.pitch = p.pitch;
  a.plane = p.plane;
  a.nplanes = p.n[0];
  a.twy = twb + p.twy;
  a.twz = twb + p.twz;
  a.st = c.st();
  // the clip counts of two rounds in a row: a block may still read the last round's when another
  // writes this one's
  a.part = c.part(r % 2 ? Ctx::PZ : Ctx::PVZ);
  a.zpart = c.part(r % 2 ? Ctx::PVZ : Ctx::PZ);
  a.nz = r == 0 ? p.ibpi : p.n[0];
  a.xpart = c.part(Ctx::PX);
  a.nx = p.xbpi;
  a.round = r;
  a.viol = viol;
  a.vstride = vstride;
  a.post = c.post;
  return p.dt == FFCZ_F32 ? launch_plane_f32(p.Ly, p.H, &a, p.n[0] * p.B, c.s)
                          : launch_plane_f64(p.Ly, p.H, &a, p.n[0] * p.B, c.s);
}

// Round r: its check, and the projections up to the next iterate.  With the plane pass the
// y-forward transform of rounds after the first is the end of the round before.
template <typename T>
hipError_t enqueue_round(const Ctx& c, int r, unsigned long long* viol, int64_t vstride, uint8_t* fmask,
                         uint32_t* smask) {
  const Plan& p = *c.p;
  unsigned long long* px = c.part(Ctx::PX);
  const char* twb = (const char*)c.twT();
  const void* twy = twb + sizeof(cx<T>) * p.twy;
  const void* twx = twb + sizeof(cx<T>) * p.twx;
  hipError_t e;
  if (p.nd == 3) {
    if (!p.planes || r == 0) {
      e = timed(PK_YFWD, r, c.s, [&] {
        return run_col<T>(p.dt, COL_FWD, p.vy, geom_y(p, p.pitch, p.plane), p, c.Z(), c.A(), twy, c.st(), px, fmask,
                          c.s);
      });
      if (e != hipSuccess) return e;
    }
    e = timed(PK_XPASS, r, c.s, [&] { return xpass_T<T>(c, c.A(), c.A(), twx, px, fmask); });
    if (e != hipSuccess) return e;
    if (p.planes) return timed(PK_ZPASS, r, c.s, [&] { return run_planes<T>(c, r, viol, vstride); });
    e = launch_ctl(c, viol, vstride);
    if (e != hipSuccess) return e;
    e = timed(PK_YINV, r, c.s, [&] {
      return run_col<T>(p.dt, COL_INV, p.vy, geom_y(p, p.pitch, p.plane), p, c.A(), c.A(), twy, c.st(), px, fmask, c.s);
    });
    if (e != hipSuccess) return e;
  } else {
    e = timed(PK_XPASS, r, c.s, [&] { return xpass_T<T>(c, c.Z(), c.A(), twx, px, fmask); });
    if (e != hipSuccess) return e;
    e = launch_ctl(c, viol, vstride);
    if (e != hipSuccess) return e;
  }
  return timed(PK_ZPASS, r, c.s, [&] { return row_T<T>(ROW_LOOP, c, c.A(), c.Z(), smask); });
}

// The check that ends the loop (converged, or at the round cap) clips inside the x-pass, but
// that clip never reaches the iterate; with edit bookkeeping its displacements went into
// the frequency edits all the same.  Repeat that check's forward transforms from Z (which
// still holds the last-axis R2C of the checked iterate) and subtract the same displacements.
template <typename T>
hipError_t enqueue_undo(const Ctx& c) {
  const Plan& p = *c.p;
  const char* twb = (const char*)c.twT();
  const void* twy = twb + sizeof(cx<T>) * p.twy;
  const void* twx = twb + sizeof(cx<T>) * p.twx;
  if (p.nd == 3) {
    hipError_t e = run_col<T>(p.dt, COL_FWD_NS, 0, geom_y(p, p.pitch, p.plane), p, c.Z(), c.A(), twy, c.st(), nullptr,
                              nullptr, c.s);
    if (e != hipSuccess) return e;
    return run_col<T>(p.dt, COL_XUNDO, 0, geom_x(p, p.pitch, p.plane), p, c.A(), nullptr, twx, c.st(), nullptr,
                      nullptr, c.s, c.facc);
  }
  return run_col<T>(p.dt, COL_XUNDO, 0, geom_x(p, p.pitch, p.plane), p, c.Z(), nullptr, twx, c.st(), nullptr,
                    nullptr, c.s, c.facc);
}

// FP64 verification: last-axis R2C of y - x (max |y - x|), then the y and x
// transforms of that spectrum with the max-reduce in the x-pass.
template <typename T>
hipError_t enqueue_verify(const Ctx& c, bool z_done) {
  const Plan& p = *c.p;
  const char* tb = (const char*)c.tw64();
  void* W = c.W();
  hipError_t e = hipSuccess;
  if (!z_done) {
    e = timed(PK_VZ, -1, c.s, [&] {
      return run_row<double, T>(1, p.dt, c.pD ? ROW_VERIFYP : ROW_VERIFY, kVerifyRowPlan, p, p.pitch64, p.plane64,
                                nullptr, W, tb + 16 * (kVerifyRowPlan == 2 ? p.twz8 : p.twz), c.st(),
                                c.part(Ctx::PVZ), nullptr, c.s);
    });
    if (e != hipSuccess) return e;
  }
  if (p.nd == 3) {
    e = timed(PK_VY, -1, c.s, [&] {
      return run_col<double>(1, COL_FWD_NS, 0, geom_y(p, p.pitch64, p.plane64), p, W, W, tb + 16 * p.twy, c.st(),
                             c.part(Ctx::PVX), nullptr, c.s);
    });
    if (e != hipSuccess) return e;
  }
  e = timed(PK_VX, -1, c.s, [&] {
    if (c.pD) {
      // bounds at the working-type spectrum's layout, the transform at the FP64 one
      const ColGeom gb = geom_x(p, p.pitch, p.plane);
      return run_col<double>(1, COL_VERIFYP, 0, geom_x(p, p.pitch64, p.plane64), p, W, W, tb + 16 * p.twx, c.st(),
                             c.part(Ctx::PVX), nullptr, c.s, nullptr, c.pD, gb.so, gb.s, p.dt == FFCZ_F64 ? 1 : 0);
    }
    return run_col<double>(1, COL_VERIFY, 0, geom_x(p, p.pitch64, p.plane64), p, W, W, tb + 16 * p.twx, c.st(),
                           c.part(Ctx::PVX), nullptr, c.s);
  });
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(stats_kernel, dim3((unsigned)p.B), dim3(1024), 0, c.s, c.st(), c.part(Ctx::PVZ), p.vzbpi,
                     c.part(Ctx::PVX), c.part(Ctx::PVX + 1), p.vxbpi);
  return hipGetLastError();
}

// Closing pass (y = x + eps, FP64 closing clamp) and, when asked, the FP64 verification.
template <typename T>
hipError_t enqueue_final(const Ctx& c, bool verify) {
  const Plan& p = *c.p;
  if (c.pD) {  // pointwise bounds: closing clamp against E_n, then the pointwise verification
    hipError_t e = timed(PK_FINAL, -1, c.s, [&] {
      return run_row<T, T>(p.dt, p.dt, ROW_FINALP, 0, p, p.pitch, p.plane, c.Z(), nullptr,
                           (const char*)c.twT() + sizeof(cx<T>) * p.twz, c.st(), c.part(Ctx::PZ), nullptr, c.s);
    });
    if (e != hipSuccess || !verify) return e;
    return enqueue_verify<T>(c, false);
  }
  if (!final_fused(p)) {
    hipError_t e = timed(PK_FINAL, -1, c.s, [&] { return row_T<T>(ROW_FINAL, c, c.Z(), nullptr, nullptr); });
    if (e != hipSuccess || !verify) return e;
    return enqueue_verify<T>(c, false);
  }
  const char* tb = (const char*)c.tw64();
  const int mode = verify ? ROW_FINALV : ROW_FINAL;
  hipError_t e = timed(PK_FINAL, -1, c.s, [&] {
    return run_row<double, T>(1, p.dt, mode, 2, p, p.pitch64, p.plane64, c.Z(), c.W(), tb + 16 * p.twz8, c.st(),
                              c.part(Ctx::PVZ), nullptr, c.s, p.pitch, p.plane);
  });
  if (e != hipSuccess || !verify) return e;
  return enqueue_verify<T>(c, true);
}

// pinned host staging (one per thread), grown on demand
struct HostBuf {
  void* p = nullptr;
  size_t n = 0;
  ~HostBuf() {
    if (p) (void)hipHostFree(p);
  }
  hipError_t reserve(size_t bytes) {
    if (bytes <= n) return hipSuccess;
    if (p) (void)hipHostFree(p);
    p = nullptr;
    n = 0;
    hipError_t e = hipHostMalloc(&p, bytes, hipHostMallocDefault);
    if (e == hipSuccess) n = bytes;
    return e;
  }
};
thread_local HostBuf g_host_state, g_host_init, g_host_misc;
// staging of the 1D members (descriptors, then their loop states), apart from the grouped members',
// which is written while copies from this one may be in flight
thread_local HostBuf g_host_sig, g_host_sigstate;

// Private streams (default priority) for the 1D members of a batch, which run beside the
// grouped members and beside one another.
struct Streams {
  // side: the 1D members of a mixed batch (else a lane); side2: the 1D members that run one block
  // each; lane1: 1D length classes beside those on the class lane 0.  With the caller's stream
  // these are four, the hardware queues of a process: streams past that share a queue and
  // wait for one another.
  hipStream_t side = nullptr, side2 = nullptr, lane1 = nullptr;
  hipEvent_t fork = nullptr, join = nullptr, fork2 = nullptr, join2 = nullptr, lfork = nullptr,
             ljoin[2] = {nullptr, nullptr};
  ~Streams() {
    for (hipStream_t q : {side, side2, lane1})
      if (q) (void)hipStreamDestroy(q);
    for (hipEvent_t ev : {fork, join, fork2, join2, lfork, ljoin[0], ljoin[1]})
      if (ev) (void)hipEventDestroy(ev);
  }
  hipError_t ready() {
    hipError_t e = hipSuccess;
    for (hipStream_t* q : {&side, &side2, &lane1})
      if (e == hipSuccess && !*q) e = hipStreamCreateWithFlags(q, hipStreamNonBlocking);
    for (hipEvent_t* ev : {&fork, &join, &fork2, &join2, &lfork, &ljoin[0], &ljoin[1]})
      if (e == hipSuccess && !*ev) e = hipEventCreateWithFlags(ev, hipEventDisableTiming);
    return e;
  }
};
// The calling thread's streams beside the stream s, on its device: a launch runs on its stream's
// device, whatever device is current, so a thread that serves several devices must not send one's
// work down another's streams.
hipError_t streams_of(hipStream_t s, Streams** out) {
  thread_local std::map<int, Streams> of;
  int dev = 0, cur = 0;
  hipError_t e = hipGetDevice(&cur);
  if (e != hipSuccess) return e;
  // (the null stream is the current device's, and so is a handle that names no stream of its own)
  if (!s || hipStreamGetDevice(s, &dev) != hipSuccess) {
    (void)hipGetLastError();
    dev = cur;
  }
  *out = &of[dev];
  if (dev == cur) return (*out)->ready();
  if ((e = hipSetDevice(dev)) != hipSuccess) return e;
  e = (*out)->ready();
  const hipError_t back = hipSetDevice(cur);
  return e != hipSuccess ? e : back;
}

// The words the control kernels post checks to: pinned host memory of the calling thread.
struct Posts : PostWords {
  ~Posts() {
    if (p) (void)hipHostFree(p);
  }
  hipError_t start(size_t words) {
    if (words > n) {
      if (p) (void)hipHostFree(p);
      p = nullptr;
      n = 0;
      const hipError_t e = hipHostMalloc((void**)&p, words * sizeof(*p), hipHostMallocMapped | hipHostMallocCoherent);
      if (e != hipSuccess) return e;
      n = words;
    }
    begin(words);
    return hipSuccess;
  }
  Post at(size_t i) const { return Post{p + i, tag}; }
};
thread_local Posts g_posts;

// Rounds of one loop, enqueued by drive() on one stream: words [w0, w0 + n) of g_posts tell
// how far its instances are.
struct RoundTask {
  hipStream_t s;
  size_t w0, n;
  std::function<hipError_t(int)> round;  // enqueue round r
  int enq = 0;
  bool done = false;
};

// Run loops to their end: round r is enqueued once check r - 1 has been posted and some instance
// goes on.  The passes between a check and the next round (the inverse transforms and the
// spatial clip) run meanwhile, so the device does not wait for the host, and the only work past
// the last check is those passes' early returns.  (Chunks of 4 rounds replayed as a hipGraph with
// one poll per chunk, measured before: 64^3 FP64, 4 rounds, 238 us, of which 3 rounds of early
// returns 30 us, two polls 30 us; a new workspace paid for a capture.)
int32_t drive(std::vector<RoundTask>& tasks, int32_t max_iter) {
  using std::chrono::microseconds;
  // captured work never runs, so nothing would be posted: refused like any wait under capture
  for (const RoundTask& t : tasks) {
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    HIPCHK(hipStreamIsCapturing(t.s, &cs));
    if (cs == hipStreamCaptureStatusNone) continue;
    HIPCHK(hipStreamSynchronize(t.s));  // an error here, which also ends the capture
    return fail(FFCZ_E_HIP, "the rounds wait for the device: not while the stream is being captured");
  }
  auto last_query = std::chrono::steady_clock::now(), since = last_query;  // since: the last round enqueued
  for (;;) {
    bool all = true, moved = false;
    for (RoundTask& t : tasks) {
      if (t.done) continue;
      int low = INT_MAX;
      for (size_t i = 0; i < t.n; ++i) {
        const PostWords::Seen v = g_posts.read(t.w0 + i);
        if (!v.done) low = std::min(low, v.checks);
      }
      if (low == INT_MAX) {
        t.done = true;
        continue;
      }
      all = false;
      if (t.enq <= low && t.enq <= max_iter) {
        HIPCHK(t.round(t.enq));
        ++t.enq;
        moved = true;
      }
    }
    if (all) return FFCZ_OK;
    const auto now = std::chrono::steady_clock::now();
    if (moved) {
      since = now;
      continue;
    }
    // rounds of small fields take tens of microseconds, which a scheduled-out thread would miss;
    // a longer wait leaves the core to whoever else is ready (a call with 0.6 s of work ahead of it
    // on its stream and a busy process on its core: half of the core each with spinning alone, less
    // than 1 % of it for this thread now)
    if (now - since > microseconds(200)) std::this_thread::yield();
    if (now - last_query > microseconds(200)) {
      // a stream that failed, or drained without posting, ends the wait
      last_query = now;
      bool idle = true;
      for (RoundTask& t : tasks) {
        if (t.done) continue;
        const hipError_t e = hipStreamQuery(t.s);
        if (e == hipErrorNotReady) {
          (void)hipGetLastError();
          idle = false;
        } else if (e != hipSuccess) {
          return fail(FFCZ_E_HIP, std::string("rounds: ") + hipGetErrorString(e));
        }
      }
      if (idle) {
        bool stuck = false;
        for (RoundTask& t : tasks) {
          if (t.done) continue;
          bool fresh = true;  // every instance posted the check of the last enqueued round, or is done
          for (size_t i = 0; i < t.n; ++i) {
            const PostWords::Seen v = g_posts.read(t.w0 + i);
            fresh = fresh && (v.done || (v.checks > 0 && v.checks >= t.enq));
          }
          if (!fresh) stuck = true;
        }
        if (stuck) return fail(FFCZ_E_HIP, "loop did not report completion (device state inconsistent)");
      }
    }
#if defined(__x86_64__)
    __builtin_ia32_pause();
#endif
  }
}

double bits_to_double(unsigned long long b) {
  double d;
  memcpy(&d, &b, 8);
  return d;
}

__global__ void zero_u64_kernel(unsigned long long* p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0ull;
}

__global__ void zero_u32_kernel(uint32_t* p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0u;
}

// ---------------------------------------------------------------------------
// Plan tuner.  Each loop pass of a plan (y-forward/inverse, x-pass, last-axis
// pass) has a few variants: tilings that compute bit-identical results and
// differ only in how many columns / rows one block owns, and for the last-axis
// passes a radix-8 stage plan.  On the first use of a pass geometry on a device
// architecture, every variant is timed on the plan's own workspace (in place on
// the scratch spectrum, before the correction starts) and the fastest is kept;
// a variant other than the default must win by 2 % (rows) or 10 % (columns).
// The table is process-wide and, when a cache path is set, read from and
// written back to a JSON file.

struct TuneEntry {
  int choice = 0;
  std::vector<float> ms;
};

struct Tuner {
  std::mutex m;
  int mode = -1;  // -1: not read yet; 0: default plans; 1: tune on a miss; 2: narrower tiles; 3: radix-8 rows
  bool loaded = false;
  std::string path;
  std::map<std::string, TuneEntry> tab;

  void init_locked() {
    if (mode >= 0) return;
    const char* e = getenv("FFCZ_AUTOTUNE");
    mode = (e && e[0] == '0') ? 0 : 1;
    const char* c = getenv("FFCZ_PLAN_CACHE");
    if (c && *c) path = c;
  }
  // Entries are one per line: "key": {"choice": N, "ms": [..]}.  Lines that do
  // not parse are ignored, so a damaged file only costs a re-tune.
  void load_locked() {
    if (loaded) return;
    loaded = true;
    if (path.empty()) return;
    FILE* f = fopen(path.c_str(), "r");
    if (!f) return;
    char line[1024];
    while (fgets(line, sizeof(line), f)) {
      const char* q0 = strchr(line, '"');
      if (!q0) continue;
      const char* q1 = strchr(q0 + 1, '"');
      if (!q1) continue;
      const char* ch = strstr(q1, "\"choice\":");
      if (!ch) continue;
      int v = -1;
      if (sscanf(ch + 9, "%d", &v) != 1 || v < 0 || v >= std::max(kColVariants, kRowVariants)) continue;
      TuneEntry te;
      te.choice = v;
      tab[std::string(q0 + 1, q1)] = te;
    }
    fclose(f);
  }
  void save_locked() {
    if (path.empty()) return;
    const std::string tmp = path + ".tmp";
    FILE* f = fopen(tmp.c_str(), "w");
    if (!f) return;
    fprintf(f, "{\n \"format\": \"ffcz tile plans 1\",\n \"entries\": {\n");
    size_t i = 0;
    for (const auto& kv : tab) {
      fprintf(f, "  \"%s\": {\"choice\": %d, \"ms\": [", kv.first.c_str(), kv.second.choice);
      for (size_t k = 0; k < kv.second.ms.size(); ++k) fprintf(f, "%s%.5f", k ? ", " : "", kv.second.ms[k]);
      fprintf(f, "]}%s\n", ++i < tab.size() ? "," : "");
    }
    fprintf(f, " }\n}\n");
    const bool ok = fclose(f) == 0;
    if (ok) rename(tmp.c_str(), path.c_str());
  }
};
Tuner g_tuner;

std::string device_arch() {
  thread_local std::map<int, std::string> names;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return "unknown";
  auto it = names.find(dev);
  if (it != names.end()) return it->second;
  hipDeviceProp_t prop;
  std::string n = "unknown";
  if (hipGetDeviceProperties(&prop, dev) == hipSuccess) n = prop.gcnArchName;
  names[dev] = n;
  return n;
}

// The variant kept for `key`; on a miss, time `launch(v)` for every variant
// (only if may_time, else the default tiles).
template <typename F>
int32_t tune_pass(const std::string& key, hipStream_t s, bool may_time, float keep, int nvar, F&& launch, int* out) {
  *out = 0;
  {
    std::lock_guard<std::mutex> g(g_tuner.m);
    g_tuner.init_locked();
    g_tuner.load_locked();
    if (g_tuner.mode == 0) return FFCZ_OK;
    if (g_tuner.mode == 2) {  // the narrower tiles
      *out = 1;
      return FFCZ_OK;
    }
    if (g_tuner.mode == 3) {  // the radix-8 last-axis plan
      *out = nvar > 2 ? 2 : 0;
      return FFCZ_OK;
    }
    if (g_tuner.mode == 4) {  // the direct (index-fastest) last-axis loop pass
      *out = nvar > 3 ? 3 : 0;
      return FFCZ_OK;
    }
    auto it = g_tuner.tab.find(key);
    if (it != g_tuner.tab.end() && it->second.choice < nvar) {
      *out = it->second.choice;
      return FFCZ_OK;
    }
  }
  if (!may_time) return FFCZ_OK;
  hipEvent_t e0, e1;
  HIPCHK(hipEventCreate(&e0));
  HIPCHK(hipEventCreate(&e1));
  TuneEntry te;
  hipError_t err = hipSuccess;
  for (int v = 0; v < nvar && err == hipSuccess; ++v) {
    err = launch(v);  // warm-up
    if (err != hipSuccess) break;
    float best = 1e30f;
    for (int rep = 0; rep < 3 && err == hipSuccess; ++rep) {
      err = hipEventRecord(e0, s);
      if (err == hipSuccess) err = launch(v);
      if (err == hipSuccess) err = hipEventRecord(e1, s);
      if (err == hipSuccess) err = hipEventSynchronize(e1);
      float ms = 0.f;
      if (err == hipSuccess) err = hipEventElapsedTime(&ms, e0, e1);
      best = std::min(best, ms);
    }
    te.ms.push_back(best);
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  HIPCHK(err);
  te.choice = 0;
  for (int v = 1; v < nvar; ++v)
    if (te.ms[v] < keep * te.ms[0] && te.ms[v] < te.ms[te.choice]) te.choice = v;
  std::lock_guard<std::mutex> g(g_tuner.m);
  g_tuner.tab[key] = te;
  g_tuner.save_locked();
  *out = te.choice;
  return FFCZ_OK;
}

// A narrower column tile reads 64-byte halves of lines whose other halves belong to
// another block (fetched again, from the last-level cache at best), so it must win clearly.
constexpr float kColKeep = 0.90f;

// Pick the loop passes' tile variants for plan p (state and twiddles already
// written; the scratch spectrum A is overwritten).  Nothing is timed while the
// stream is being captured or masks are recorded (the loop kernels would write
// mask planes); mask recording also keeps the default x-pass tiles, whose
// width the 1-bit mask words assume.
// Table key of a plan's last-axis loop pass.
std::string tune_key_z(const Plan& p) {
  char buf[256];
  snprintf(buf, sizeof(buf), "%s z H=%d rows=%lld", (device_arch() + (p.dt == FFCZ_F32 ? " f32" : " f64")).c_str(), p.H,
           (long long)(p.nrows * p.B));
  return buf;
}

// no_time: take the table's decisions (or the defaults) without timing anything.
template <typename T>
int32_t tune_plan(Plan& p, char* ws, hipStream_t s, bool rec, bool no_time = false) {
  const std::string pre = device_arch() + (p.dt == FFCZ_F32 ? " f32" : " f64");
  char buf[256];
  int vy = 0, vx = 0, vz = 0;
  Ctx c{&p, ws, s};
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  HIPCHK(hipStreamIsCapturing(s, &cs));
  const bool may_time = !rec && !no_time && cs == hipStreamCaptureStatusNone;
  const char* twb = (const char*)c.twT();
  if (p.nd == 3 && p.Ly >= 64) {
    snprintf(buf, sizeof(buf), "%s y L=%d cols=%lld outer=%lld", pre.c_str(), p.Ly, (long long)p.ncols,
             (long long)p.n[0]);
    int32_t r = tune_pass(buf, s, may_time, kColKeep, kColVariants, [&](int v) {
      return run_col<T>(p.dt, COL_FWD, v, geom_y(p, p.pitch, p.plane), p, c.A(), c.A(), twb + sizeof(cx<T>) * p.twy,
                        c.st(), c.part(Ctx::PX), nullptr, s);
    }, &vy);
    if (r != FFCZ_OK) return r;
  }
  if (p.nd >= 2 && p.Lx >= 64 && !rec) {
    snprintf(buf, sizeof(buf), "%s x L=%d cols=%lld outer=%lld B=%lld", pre.c_str(), p.Lx, (long long)p.ncols,
             (long long)(p.nd == 3 ? p.n[1] : 1), (long long)p.B);
    int32_t r = tune_pass(buf, s, may_time, kColKeep, kColVariants, [&](int v) {
      Plan q = p;
      set_variants(q, q.vy, v, q.vz);
      return run_col<T>(p.dt, COL_XPASS, v, geom_x(q, q.pitch, q.plane), q, c.A(), c.A(), twb + sizeof(cx<T>) * p.twx,
                        c.st(), c.part(Ctx::PX), nullptr, s);
    }, &vx);
    if (r != FFCZ_OK) return r;
  }
  if (p.H >= 64) {
    int32_t r = tune_pass(tune_key_z(p), s, may_time, 0.98f, kRowVariants, [&](int v) {
      return run_row<T, T>(p.dt, p.dt, ROW_LOOP, v, p, p.pitch, p.plane, c.A(), c.A(),
                           twb + sizeof(cx<T>) * (v == 2 ? p.twz8 : p.twz), c.st(),
                           c.part(Ctx::PZ), nullptr, s);
    }, &vz);
    if (r != FFCZ_OK) return r;
    if (rec) vz = masked_variant(p, vz);
  }
  set_variants(p, vy, vx, vz);
  return FFCZ_OK;
}

// Whether a field's rounds run on the plane pass: one block does a whole plane, so a plane must
// either be small (a few us a block) or come in numbers that keep the chip busy.  And with enough
// planes to fill the chip several times over, what counts is each pass's rate, not its launch and
// its latency: with rows of 64 entries and more the separate passes' is the higher one (longer y
// transforms make up for it in FP64 planes of 128 KB).  20 rounds, separate -> plane pass, us
// (MI355X; n0 x n1 x n2):
//   up to 32 KB  64 x 64 x 64 FP64 616 -> 414, 2 x 64 x 64 FP32 497 -> 306, 64 x 64 x 128 FP32 604 -> 460;
//                512 x 64 x 128 FP32 1119 -> 1031, but 1024: 1755 -> 1806 and 2048: 3107 -> 3433;
//                1024 x 32 x 128 FP64 1713 -> 1846; 2048 x 32 x 256 FP32 2890 -> 3358
//   64 KB        64 x 256 x 64 FP32 757 -> 699, but 16: 590 -> 626; 64 x 64 x 128 FP64 723 -> 643;
//                512 x 128 x 128 FP32 1621 -> 1480, but 2048: 6151 -> 6382; 1024 x 32 x 256 FP64 2822 -> 2924
//   128 KB FP32  256 x 512 x 64 1790 -> 1611, but 128: 1182 -> 1192; 256 x 128 x 256 1458 -> 1363,
//                but 512: 2448 -> 2488 and 1024: 5061 -> 5195; 512 x 256 x 128 2701 -> 2620
//   128 KB FP64  128 x 128 x 128 1137 -> 1074, but 64: 958 -> 965; 1024 x 64 x 256 5021 -> 4711
bool plane_rule(const Plan& p) {
  const int64_t planes = p.n[0] * p.B;
  const bool f32 = p.dt == FFCZ_F32;
  if (p.nd != 3 || planes > p.pmax) return false;
  if (!(f32 ? plane_fits<float>(p.Ly, p.H) : plane_fits<double>(p.Ly, p.H))) return false;
  const int64_t kb = (int64_t)p.Ly * p.H * (f32 ? 8 : 16) / 1024;
  if (kb > 32 && planes < (kb <= 64 ? 64 : f32 ? 256 : 128)) return false;
  if (p.Ly > 16 && p.H >= 64 && planes >= 1024 && (f32 || kb <= 64)) return false;
  if (f32 && kb > 64 && p.H >= 128 && planes >= 512) return false;
  std::lock_guard<std::mutex> g(g_tuner.m);
  g_tuner.init_locked();
  return g_tuner.mode == 1;  // the other modes ask for the separate passes' plans
}

// Tune a group's passes ahead of a mixed batch, before the 1D members start on
// the side stream (their work would disturb the timings): a neutral state (loop
// not done, no masks) and the twiddles are written, then tune_plan runs on the
// group's own workspace.  The decisions land in the process-wide table.
template <typename T>
int32_t pretune_group(const Plan& p0, char* ws, hipStream_t s) {
  Plan p = p0;
  Ctx c{&p, ws, s};
  StateInit one;
  memset(&one, 0, sizeof(one));
  one.max_iter = 1;
  HIPCHK(run_setup(c, nullptr, one, nullptr, 0));
  return tune_plan<T>(p, ws, s, false);
}

// Edit bookkeeping of an encoder call (null for a plain correction).
struct EditCfg {
  void* sacc;     // spatial accumulators: N values of the working type, C order
  void* facc;     // frequency accumulators: laid out as the spectrum Z
  bool derive;    // shrinks from x on the device; else mu_s / mu_f below
  double q;       // safety 2^-m (derive)
  double mu_s, mu_f;
  bool want_y;    // close y = x + eps (and verify it when asked)
  unsigned long long* amax;  // kUlpSlots partial slots of max |x| (derive)
  double* mu_s_out;          // host: the spatial shrink in use, read back with the state
};

// Workspace of the encoder and decoder: the plan's, then the accumulators and the
// coding kernels' block offsets.
struct EditLayout {
  int64_t ncs = 0, ncf = 0;  // spatial and frequency coordinates
  int64_t nbs = 0, nbf = 0;  // coding blocks of each set
  size_t off_S = 0, off_F = 0, off_offs = 0, off_offf = 0, off_tot = 0, off_amax = 0, bytes = 0;
  int64_t spec_reals = 0;    // working-type reals of one spectrum buffer (padding included)
};

EditLayout edit_layout(const Plan& p) {
  EditLayout L;
  const size_t ts = p.dt == FFCZ_F32 ? 4 : 8;
  L.ncs = p.N * p.B;
  L.ncf = 2 * p.nrows * p.ncols * p.B;
  L.nbs = (L.ncs + kEditBlockCoords - 1) / kEditBlockCoords;
  L.nbf = (L.ncf + kEditBlockCoords - 1) / kEditBlockCoords;
  const int64_t rpp = p.nd == 3 ? p.n[1] : p.nrows;
  L.spec_reals = 2 * p.B * (p.nrows / rpp) * p.plane;
  size_t off = align_up(p.bytes, 256);
  L.off_S = off;
  off = align_up(off + ts * (size_t)L.ncs, 256);
  L.off_F = off;
  off = align_up(off + ts * (size_t)L.spec_reals, 256);
  L.off_offs = off;
  off = align_up(off + 8 * (size_t)std::max<int64_t>(1, L.nbs), 256);
  L.off_offf = off;
  off = align_up(off + 8 * (size_t)std::max<int64_t>(1, L.nbf), 256);
  L.off_tot = off;  // two totals and the status word
  off = align_up(off + 8 * 4, 256);
  L.off_amax = off;
  off = align_up(off + 8 * (size_t)kUlpSlots, 256);
  L.bytes = off;
  return L;
}

// Pointwise bounds of a ffcz_correct_bounds call (null for scalar bounds).
struct BoundsCfg {
  const void* pE;               // E_n (caller's device array, field dtype) or null: the scalar E
  const void* dre;              // D^Re_k (or the disk's D_k), half-spectrum C order, or null
  const void* dim;              // D^Im_k or null (then D^Re_k, or the scalar)
  double sre, sim;              // scalar spectral bounds where the arrays are null
  int disk;
  void* pD;                     // workspace: the bound pairs laid out as the spectrum
  unsigned long long* minpart;  // workspace: kMinSlots block minima
  unsigned long long* bad;      // workspace: invalid-entry counter
};

// Workspace of ffcz_correct_bounds and ffcz_power_spectrum_bounds beyond the plan's: the bound
// pairs, block minima and a counter; for the power-spectrum bound the per-block shell sums and the
// shell bounds.
struct BoundsLayout {
  size_t off_D = 0, off_min = 0, off_bad = 0, off_shell = 0, off_bins = 0, bytes = 0;
  int nb = 0;   // shells
  int nsb = 0;  // shell-sum blocks
};

BoundsLayout bounds_layout(const Plan& p) {
  BoundsLayout L;
  const size_t ts = p.dt == FFCZ_F32 ? 4 : 8;
  double kmax2 = 0.0;
  for (int i = 0; i < p.nd; ++i) kmax2 += (double)(p.n[i] / 2) * (double)(p.n[i] / 2);
  L.nb = (int)std::lrint(std::sqrt(kmax2)) + 1;
  const int64_t M = p.nrows * p.ncols;
  L.nsb = (int)std::max<int64_t>(1, std::min<int64_t>(256, (M + 4095) / 4096));
  const int64_t rpp = p.nd == 3 ? p.n[1] : p.nrows;
  size_t off = align_up(p.bytes, 256);
  L.off_D = off;
  off = align_up(off + 2 * ts * (size_t)(p.nrows / rpp) * (size_t)p.plane, 256);
  L.off_min = off;
  off = align_up(off + 8 * (size_t)kMinSlots, 256);
  L.off_bad = off;
  off = align_up(off + 8, 256);
  L.off_shell = off;
  off = align_up(off + 8 * 3 * (size_t)L.nsb * (size_t)L.nb, 256);
  L.off_bins = off;
  off = align_up(off + 8 * (size_t)L.nb, 256);
  L.bytes = off;
  return L;
}

// One correction over the B instances of a plan.  inst[b] supplies pointers and
// bounds, mus[b] the margins; mus null (one FP32 instance) derives mu from x on
// the device, between the state set-up and the first pass.
// host_state: when given (one entry per instance, ordinary host memory), the call
// allocates nothing: the loop state is read back into it, the rounds run in polled chunks
// and the tile plans come from the table or the defaults.
// One group's correction (a plan over B same-shape instances) in phases: begin (set-up through
// the first last-axis transform, on the call's stream), the rounds (driven from here, or with
// other work by the mixed-batch loop), end (closing pass, verification, statistics).  Holds a Ctx that points at its own Plan: neither copied nor moved.
template <typename T>
struct GroupRun {
  Plan p;
  Ctx c{nullptr, nullptr, nullptr};
  const ffcz_instance* inst = nullptr;
  const double* mus = nullptr;
  int32_t max_iter = 0;
  ffcz_options o{};
  DevState* host_state = nullptr;  // the no-allocation form's host copy of the state (else null)
  const EditCfg* ed = nullptr;
  const BoundsCfg* bc = nullptr;
  bool no_alloc = false, rec = false;
  unsigned long long* viol = nullptr;
  int64_t vstr = 0;
  uint32_t* smask = nullptr;
  uint8_t* fmask = nullptr;
  int chunk = 4;

  GroupRun() = default;
  GroupRun(const GroupRun&) = delete;
  GroupRun& operator=(const GroupRun&) = delete;

  int32_t begin(const Plan& p0, const ffcz_instance* inst_, const double* mus_, int32_t max_iter_,
                const ffcz_options& o_, char* ws, hipStream_t s, DevState* host_state_, const EditCfg* ed_,
                const BoundsCfg* bc_) {
    inst = inst_;
    mus = mus_;
    max_iter = max_iter_;
    o = o_;
    host_state = host_state_;
    ed = ed_;
    bc = bc_;
    no_alloc = host_state != nullptr;
    p = p0;
    c = Ctx{&p, ws, s};
    if (ed) {
      c.sacc = ed->sacc;
      c.facc = ed->facc;
    }
    if (bc) c.pD = bc->pD;
    const int64_t vstride = max_iter + 2;
    const bool user_viol = o.viol_per_round && p.B == 1;
    viol = user_viol ? (unsigned long long*)o.viol_per_round : c.viol();
    vstr = user_viol ? 0 : vstride;
    rec = o.masks_out != nullptr && p.B == 1;
    smask = rec ? (uint32_t*)o.masks_out : nullptr;
    fmask = rec ? (uint8_t*)o.masks_out + (size_t)(max_iter + 1) * p.s_plane_bytes : nullptr;
    chunk = o.graph_chunk > 0 ? o.graph_chunk : 4;

    auto fill = [&](int64_t b) {
      StateInit si;
      memset(&si, 0, sizeof(si));
      si.E = inst[b].eps_s;
      const double mu = mus ? mus[b] : 0.0;  // without mus, margin_kernel rewrites the mu-dependent fields
      si.Ep = inst[b].eps_s * (1.0 - mu);
      si.Delta = inst[b].delta_f;
      spectral_thresholds(p.dt, inst[b].delta_f, mu, &si.Dc, &si.Dp);
      si.inv_n = 1.0 / (double)p.N;
      si.mu = mu;
      if (ed && !ed->derive) {  // the encoder's given shrinks
        si.mu = ed->mu_f;
        si.mu_s = ed->mu_s;
        si.Ep = inst[b].eps_s * (1.0 - ed->mu_s);
        si.Dc = inst[b].delta_f * (1.0 - ed->mu_f);
        si.Dp = inst[b].delta_f * (1.0 - 2.0 * ed->mu_f);
      }
      if (bc) {
        si.pE = bc->pE;
        si.pD = bc->pD;
        si.disk = bc->disk;
      }
      si.max_iter = max_iter;
      si.fixed = o.fixed_iterations ? 1 : 0;
      si.record_masks = rec ? 1 : 0;
      si.px = inst[b].x_orig;
      si.pxb = inst[b].x_base;
      si.py = inst[b].x_out;
      return si;
    };
    const StateInit* arr = nullptr;
    StateInit one = fill(0);
    if (p.B > 1) {
      HIPCHK(g_host_init.reserve(sizeof(StateInit) * p.B));
      StateInit* h = (StateInit*)g_host_init.p;
      for (int64_t b = 0; b < p.B; ++b) h[b] = fill(b);
      arr = (const StateInit*)(ws + p.off_init);
      HIPCHK(hipMemcpyAsync((void*)arr, h, sizeof(StateInit) * p.B, hipMemcpyHostToDevice, s));
    }
    const int64_t nviol = user_viol ? (int64_t)max_iter + 1 : vstride * p.B;
    // an FP32 field whose margin is not given: its ulp partials with the set-up
    const MarginJob mjob{(const float*)inst[0].x_orig, p.N, inst[0].delta_f, 0};
    const bool from_x = p.B == 1 && p.dt == FFCZ_F32 && (bc ? !(mus && mus[0] > 0.0) : ed ? ed->derive : !mus);
    HIPCHK(run_setup(c, arr, one, viol, nviol, from_x ? &mjob : nullptr));
    if (bc) {
      // the bound pairs into the spectrum layout, their checks and minimum, then mu and the factors
      if (p.B != 1) return fail(FFCZ_E_INVALID, "pointwise bounds take one instance");
      hipLaunchKernelGGL(zero_u64_kernel, dim3(1), dim3(64), 0, s, bc->bad, (int64_t)1);
      HIPCHK(hipGetLastError());
      const int64_t M = p.nrows * p.ncols;
      const int nmin = (int)std::max<int64_t>(1, std::min<int64_t>(kMinSlots, (M + 255) / 256));
      const SpecGeom g{p.nrows, (int32_t)p.ncols, p.lg_rpp, p.pitch, p.plane};
      hipLaunchKernelGGL(bounds_setup_kernel<T>, dim3((unsigned)nmin), dim3(256), 0, s, (const T*)bc->dre,
                         (const T*)bc->dim, bc->sre, bc->sim, (cx<T>*)bc->pD, M, g, bc->minpart, bc->bad);
      HIPCHK(hipGetLastError());
      if (bc->pE) {
        const int nbe = (int)std::max<int64_t>(1, std::min<int64_t>(1024, (p.N + 255) / 256));
        hipLaunchKernelGGL(spatial_check_kernel<T>, dim3((unsigned)nbe), dim3(256), 0, s, (const T*)bc->pE, p.N,
                           bc->bad);
        HIPCHK(hipGetLastError());
      }
      double* slots = (double*)(ws + p.off_ulp);
      const double mu_given = mus ? mus[0] : 0.0;
      hipLaunchKernelGGL(bounds_margin_kernel, dim3(1), dim3(256), 0, s, (const double*)slots,
                         (const unsigned long long*)bc->minpart, nmin, p.N, (int)p.dt, bc->disk, mu_given, c.st());
      HIPCHK(hipGetLastError());
      unsigned long long nbad = 0;
      HIPCHK(hipMemcpyAsync(&nbad, bc->bad, sizeof(nbad), hipMemcpyDeviceToHost, s));
      HIPCHK(hipStreamSynchronize(s));
      if (nbad) return fail(FFCZ_E_INVALID, "bound arrays must hold finite values >= 0 (" + std::to_string(nbad) +
                                                " entries do not)");
    } else if (ed && ed->derive) {
      // the encoder's shrinks from x (ulp partials for the FP32 output margin, max |x|)
      if (p.B != 1) return fail(FFCZ_E_INVALID, "the encoder takes one instance");
      const int nsl = ulp_slots(p.N);
      double* slots = (double*)(ws + p.off_ulp);
      if (p.dt == FFCZ_F32) {
        hipLaunchKernelGGL(absmax_part_kernel<float>, dim3((unsigned)nsl), dim3(256), 0, s,
                           (const float*)inst[0].x_orig, p.N, ed->amax);
      } else {
        hipLaunchKernelGGL(absmax_part_kernel<double>, dim3((unsigned)nsl), dim3(256), 0, s,
                           (const double*)inst[0].x_orig, p.N, ed->amax);
      }
      HIPCHK(hipGetLastError());
      hipLaunchKernelGGL(encode_margin_kernel, dim3(1), dim3(256), 0, s, (const double*)slots,
                         (const unsigned long long*)ed->amax, p.N, (int)p.dt, ed->q, c.st());
      HIPCHK(hipGetLastError());
    } else if (!mus) {
      if (p.B != 1 || p.dt != FFCZ_F32) return fail(FFCZ_E_INVALID, "device margin needs one FP32 instance");
      hipLaunchKernelGGL(margin_kernel, dim3(1), dim3(256), 0, s, (const double*)(ws + p.off_ulp), mjob,
                         (const MarginJob*)nullptr, (int)p.dt, (double*)nullptr, c.st());
      HIPCHK(hipGetLastError());
    }
    if (bc) {
      set_variants(p, 0, 0, 0);  // the pointwise passes exist for the default tiles only
    } else if (ed) {
      // edit bookkeeping runs on the default tiles; the frequency accumulators start at zero
      set_variants(p, 0, 0, 0);
      const int64_t nr = edit_layout(p).spec_reals;
      hipLaunchKernelGGL(zero_fill_kernel<T>, dim3((unsigned)((nr + 4096 / sizeof(T) - 1) / (4096 / sizeof(T)))),
                         dim3(256), 0, s, (T*)ed->facc, nr);
      HIPCHK(hipGetLastError());
    } else {
      const int32_t tr = tune_plan<T>(p, ws, s, rec, no_alloc);
      if (tr != FFCZ_OK) return tr;
      if (!rec && plane_rule(p)) {
        p.planes = true;
        p.zbpi = p.n[0];
      }
    }
    HIPCHK(timed(PK_INIT, -1, s, [&] { return row_T<T>(ROW_INIT, c, nullptr, c.Z(), smask); }));
    return FFCZ_OK;
  }

  hipError_t round(int r) const { return enqueue_round<T>(c, r, viol, vstr, fmask, smask); }

  // The rounds as a task of drive(), checks posted from word w0 on.
  RoundTask task(size_t w0) {
    c.post = g_posts.at(w0);
    return RoundTask{c.s, w0, (size_t)p.B, [this](int r) { return round(r); }};
  }

  // The host copy of the instances' states (the no-allocation form brings its own).
  int32_t host_states(DevState** hs) {
    if (!no_alloc) HIPCHK(g_host_state.reserve(sizeof(DevState) * p.B));
    *hs = no_alloc ? host_state : (DevState*)g_host_state.p;
    return FFCZ_OK;
  }

  // The rounds, driven from here: fixed rounds enqueued at once; else round by round as checks are
  // posted (drive), or, on request and in the no-allocation form, in chunks with one poll of the
  // done-flags per chunk.
  int32_t loop() {
    const hipStream_t s = c.s;
    if (o.fixed_iterations) {
      // exactly max_iter blocks plus the final check: no polling needed
      for (int r = 0; r <= max_iter; ++r) HIPCHK(round(r));
      return FFCZ_OK;
    }
    if (o.use_graph && !no_alloc) {
      HIPCHK(g_posts.start((size_t)p.B));
      std::vector<RoundTask> t{task(0)};
      return drive(t, max_iter);
    }
    DevState* hs = nullptr;
    int32_t hr = host_states(&hs);
    if (hr != FFCZ_OK) return hr;
    for (int enq = 0;;) {
      for (int r = 0; r < chunk; ++r) HIPCHK(round(enq + r));
      enq += chunk;
      HIPCHK(hipMemcpyAsync(hs, c.st(), sizeof(DevState) * p.B, hipMemcpyDeviceToHost, s));
      HIPCHK(hipStreamSynchronize(s));
      bool all = true;
      for (int64_t b = 0; b < p.B; ++b) all = all && hs[b].done;
      if (all) break;
      if (enq > max_iter + 2 * chunk + 2)
        return fail(FFCZ_E_HIP, "loop did not report completion (device state inconsistent)");
    }
    return FFCZ_OK;
  }

  // After the rounds: the closing pass and verification, then (unless nothing is reported)
  // the instances' statistics and statuses.
  int32_t end(ffcz_stats* stats, int32_t* status) {
    DevState* hs = nullptr;
    int32_t hr = host_states(&hs);
    if (hr != FFCZ_OK) return hr;
    // asynchronous only when nothing is reported: fixed rounds, no statistics, no verification
    const bool sync_needed = !(o.fixed_iterations && stats == nullptr && !o.verify_fp64);
    if (ed) HIPCHK(enqueue_undo<T>(c));
    if (!ed || ed->want_y) HIPCHK(enqueue_final<T>(c, o.verify_fp64 != 0));
    if (!sync_needed) {
      prof_settle(max_iter);
      for (int64_t b = 0; b < p.B; ++b) status[b] = FFCZ_OK;
      return FFCZ_OK;
    }
    HIPCHK(hipMemcpyAsync(hs, c.st(), sizeof(DevState) * p.B, hipMemcpyDeviceToHost, c.s));
    HIPCHK(hipStreamSynchronize(c.s));
    int maxr = 0;
    for (int64_t b = 0; b < p.B; ++b) maxr = std::max(maxr, hs[b].round);
    prof_settle(maxr);
    if (ed && ed->mu_s_out) *ed->mu_s_out = hs[0].mu_s;
    for (int64_t b = 0; b < p.B; ++b) {
      const DevState& h = hs[b];
      const double ms = bits_to_double(h.max_spatial_bits), mf = bits_to_double(h.max_spectral_bits);
      if (stats) {
        ffcz_stats& st = stats[b];
        memset(&st, 0, sizeof(st));
        st.rounds = h.round;
        st.converged = h.converged;
        st.f_viol_initial = (int64_t)h.v_first;
        st.f_viol_final = (int64_t)h.v_last;
        st.s_clipped_total = (int64_t)h.s_clipped_total;
        st.s_guard = (int64_t)h.s_guard;
        st.nonfinite = (int64_t)h.nonfinite;
        st.max_spatial_err = o.verify_fp64 ? ms : NAN;
        st.max_spectral_err = o.verify_fp64 ? mf : NAN;
        st.spectral_viol = (int64_t)h.spectral_viol;
        st.margin_used = h.mu;
      }
      int32_t r = FFCZ_OK;
      if (h.nonfinite) r = FFCZ_E_NONFINITE;
      else if (!h.converged && !o.fixed_iterations) r = FFCZ_NOT_CONVERGED;
      else if (o.verify_fp64 && bc && (!(ms <= 1.0) || !(mf <= 1.0) || h.spectral_viol)) r = FFCZ_VERIFY_FAILED;
      else if (o.verify_fp64 && !bc && (!(ms <= inst[b].eps_s) || !(mf <= inst[b].delta_f))) r = FFCZ_VERIFY_FAILED;
      status[b] = r;
    }
    return FFCZ_OK;
  }
};

template <typename T>
int32_t correct_group(const Plan& p0, const ffcz_instance* inst, const double* mus, int32_t max_iter,
                      const ffcz_options& o, char* ws, hipStream_t s, ffcz_stats* stats, int32_t* status,
                      DevState* host_state = nullptr, const EditCfg* ed = nullptr,
                      const BoundsCfg* bc = nullptr) {
  GroupRun<T> g;
  int32_t r = g.begin(p0, inst, mus, max_iter, o, ws, s, host_state, ed, bc);
  if (r != FFCZ_OK) return r;
  r = g.loop();
  if (r != FFCZ_OK) return r;
  return g.end(stats, status);
}

template <typename T>
int32_t backward_impl(const Plan& p, int32_t rounds, const void* masks, const void* gy, void* gb, void* ws,
                      hipStream_t s) {
  Ctx c{&p, (char*)ws, s};
  StateInit si;
  memset(&si, 0, sizeof(si));
  si.inv_n = 1.0 / (double)p.N;
  si.max_iter = rounds;
  si.pxb = gy;
  si.py = gb;
  HIPCHK(run_setup(c, nullptr, si, nullptr, 0));
  const char* mb = (const char*)masks;
  auto splane = [&](int k) { return (uint32_t*)(mb + (size_t)k * p.s_plane_bytes); };
  auto fplane = [&](int k) {
    return (uint8_t*)(mb + (size_t)(rounds + 1) * p.s_plane_bytes + (size_t)(k - 1) * 2 * p.f_plane_bytes);
  };
  const char* twb = (const char*)c.twT();
  const void* twy = twb + sizeof(cx<T>) * p.twy;
  const void* twx = twb + sizeof(cx<T>) * p.twx;
  if (rounds == 0) {
    // y = x + M_s^0 (x_hat - x): the gradient is the guard mask times dL/dy (applied twice; masks are idempotent)
    HIPCHK(row_T<T>(ROW_BINIT, c, nullptr, c.Z(), splane(0)));
    HIPCHK(row_T<T>(ROW_BFINAL, c, c.Z(), nullptr, splane(0)));
    return FFCZ_OK;
  }
  HIPCHK(timed(PK_BZ, -1, s, [&] { return row_T<T>(ROW_BINIT, c, nullptr, c.Z(), splane(rounds)); }));
  for (int k = rounds; k >= 1; --k) {
    if (p.nd == 3)
      HIPCHK(timed(PK_BY, -1, s, [&] {
        return run_col<T>(p.dt, COL_FWD_NS, 0, geom_y(p, p.pitch, p.plane), p, c.Z(), c.Z(), twy, c.st(), nullptr, nullptr, s);
      }));
    HIPCHK(timed(PK_BX, -1, s, [&] {
      return run_col<T>(p.dt, COL_XBACK, 0, geom_x(p, p.pitch, p.plane), p, c.Z(), c.Z(), twx, c.st(), nullptr, fplane(k), s);
    }));
    if (p.nd == 3)
      HIPCHK(timed(PK_BY, -1, s, [&] {
        return run_col<T>(p.dt, COL_INV_NS, 0, geom_y(p, p.pitch, p.plane), p, c.Z(), c.Z(), twy, c.st(), nullptr, nullptr, s);
      }));
    if (k > 1) HIPCHK(timed(PK_BZ, -1, s, [&] { return row_T<T>(ROW_BLOOP, c, c.Z(), c.Z(), splane(k - 1)); }));
    else HIPCHK(timed(PK_BZ, -1, s, [&] { return row_T<T>(ROW_BFINAL, c, c.Z(), nullptr, splane(0)); }));
  }
  return FFCZ_OK;
}

// ---------------------------------------------------------------------------
// 1D batch members: one block per signal (kernels_sig.hpp)


struct SigPlan {
  int dt = 0;
  int64_t L = 0;
  int blue = 0;
  int lgMc = 0;
  size_t conv64 = 0, btab = 0, btab64 = 0, btabi = 0, chirp = 0, chirp64 = 0, eps = 0, bytes = 0;  // offsets in the signal block
};

SigPlan sig_plan(int dt, int64_t L) {
  SigPlan s;
  s.dt = dt;
  s.L = L;
  s.blue = (is_pow2(L) && L >= 4) ? 0 : 1;  // direct four-step needs Mc = L >= 4
  // Bluestein over the half spectrum: Mc >= L + K - 1 with K = floor(L/2) + 1
  s.lgMc = s.blue ? ceil_lg(L + L / 2) : ceil_lg(L);
  if (s.lgMc < 2) s.lgMc = 2;
  const size_t Mc = (size_t)1 << s.lgMc;
  size_t off = 0;
  s.conv64 = off;
  off = align_up(off + 16 * Mc, 256);
  if (s.blue) {
    s.btab64 = off;
    off = align_up(off + 16 * Mc, 256);
    s.chirp64 = off;
    off = align_up(off + 16 * (size_t)L, 256);
    if (dt == FFCZ_F32) {
      s.btab = off;
      off = align_up(off + 8 * Mc, 256);
      s.chirp = off;
      off = align_up(off + 8 * (size_t)L, 256);
    } else {
      s.btab = s.btab64;
      s.chirp = s.chirp64;
    }
    s.btabi = off;  // the reflected table, in the loop's working type
    off = align_up(off + (dt == FFCZ_F32 ? 8 : 16) * Mc, 256);
  }
  s.eps = off;
  off = align_up(off + (dt == FFCZ_F32 ? 4 : 8) * (size_t)L, 256);
  s.bytes = off;
  return s;
}

// four-step tables of one convolution length: working type and FP64, both layouts
struct McTabs {
  size_t tw4, tw4r, twa, twb, tw4_64, tw4r_64, twa_64, twb_64, bytes;
};

int sig_ma(int lgMc) { return 1 << ((lgMc + 1) / 2); }

McTabs mc_tabs(int dt, int lgMc) {
  const int MA = sig_ma(lgMc), MB = (1 << lgMc) / MA;
  const size_t Mc = (size_t)1 << lgMc;
  const size_t cs = dt == FFCZ_F32 ? 8 : 16;
  McTabs t;
  size_t off = 0;
  t.tw4 = off;
  off = align_up(off + cs * Mc, 256);
  t.tw4r = off;
  off = align_up(off + cs * Mc, 256);
  t.twa = off;
  off = align_up(off + cs * (host_twsize(MA, pick_E(MA)) + 1), 256);
  t.twb = off;
  off = align_up(off + cs * (host_twsize(MB, pick_E(MB)) + 1), 256);
  t.tw4_64 = off;
  off = align_up(off + 16 * Mc, 256);
  t.tw4r_64 = off;
  off = align_up(off + 16 * Mc, 256);
  t.twa_64 = off;
  off = align_up(off + 16 * (host_twsize(MA, pick_E(MA)) + 1), 256);
  t.twb_64 = off;
  off = align_up(off + 16 * (host_twsize(MB, pick_E(MB)) + 1), 256);
  t.bytes = off;
  return t;
}

// The four-step tables of every length class of a call, in one launch (bound by its own start:
// 2^20 entries of all classes take about 10 us, where a launch per table and precision, 4 per
// class, took about 10 us each).  Blocks [first, next class's first) serve a class: entry i < Mc
// is W_Mc^{n1 k2} in the column layout [k2][n1] and in the row-pass layout of the sig kernel,
// the rest are the stage twiddles of its two transform lengths.  Each value is computed once in
// FP64 and stored in FP64 and in the working type.  The grid's last blocks clear the 1D
// members' loop states.
struct TabClass {
  char* base;
  McTabs t;
  int32_t lgMc, MA, RR;
  int32_t first;  // first block
};
struct TabClasses {
  TabClass c[20];
  int32_t n, dbl;
  unsigned long long* zero;
  int64_t nzero;
  int32_t zfirst;  // first clearing block
};

__global__ void __launch_bounds__(256) sig_tables_kernel(TabClasses J) {
  if ((int)blockIdx.x >= J.zfirst) {
    const int64_t i = (int64_t)((int)blockIdx.x - J.zfirst) * 256 + threadIdx.x;
    if (i < J.nzero) J.zero[i] = 0ull;
    return;
  }
  int k = 0;
  while (k + 1 < J.n && (int)blockIdx.x >= J.c[k + 1].first) ++k;
  const TabClass& c = J.c[k];
  const int64_t Mc = (int64_t)1 << c.lgMc, i = (int64_t)((int)blockIdx.x - c.first) * 256 + threadIdx.x;
  const int MA = c.MA, MB = (int)(Mc / MA);
  double sn, cs;
  size_t o0, o1, o0_64, o1_64;  // byte offsets of the tables an entry goes to
  int64_t e0, e1;               // and its indices there
  if (i < Mc) {
    const int64_t k2 = i / MA, n1 = i % MA;
    const int64_t r = (n1 * k2) & (Mc - 1);
    sincospi(-2.0 * (double)r / (double)Mc, &sn, &cs);
    e0 = i;
    e1 = ((k2 / c.RR) * MA + n1) * c.RR + (k2 % c.RR);
    o0 = c.t.tw4;
    o1 = c.t.tw4r;
    o0_64 = c.t.tw4_64;
    o1_64 = c.t.tw4r_64;
  } else {
    // stage twiddle e of length L: stage of span ns owns ns (E - 1) entries (host_twsize)
    const int ta = host_twsize(MA, pick_E(MA)), tb = host_twsize(MB, pick_E(MB));
    int64_t e = i - Mc;
    const bool second = e >= ta;
    if (second) e -= ta;
    if (second && e >= tb) return;
    const int L = second ? MB : MA, E = pick_E(L);
    const int lgE = ilog2c(E), a = ilog2c(L) / lgE;
    const int r0 = L >> (a * lgE);
    int64_t ns = r0 > 1 ? r0 : 1, off = 0;
    for (int t = 0; t < a; ++t, ns *= E) {
      if (ns == 1) continue;
      const int64_t own = ns * (E - 1);
      if (e < off + own) break;
      off += own;
    }
    const int64_t loc = e - off, m = loc / (E - 1), r = loc % (E - 1) + 1;
    sincospi(-2.0 * (double)(m * r) / ((double)ns * E), &sn, &cs);
    e0 = e1 = e;
    o0 = o1 = second ? c.t.twb : c.t.twa;
    o0_64 = o1_64 = second ? c.t.twb_64 : c.t.twa_64;
  }
  const cx<double> w{cs, sn};
  ((cx<double>*)(c.base + o0_64))[e0] = w;
  ((cx<double>*)(c.base + o1_64))[e1] = w;
  if (J.dbl) {
    ((cx<double>*)(c.base + o0))[e0] = w;
    ((cx<double>*)(c.base + o1))[e1] = w;
  } else {
    const cx<float> f{__double2float_rn(cs), __double2float_rn(sn)};
    ((cx<float>*)(c.base + o0))[e0] = f;
    ((cx<float>*)(c.base + o1))[e1] = f;
  }
}

// Layout of the batched workspace

struct BatchPlan {
  int dt = 0;
  std::vector<int> sig_ids;                 // 1D members
  std::vector<SigPlan> sigs;
  std::map<int, std::vector<int>> by_mc;    // lgMc -> positions in sig_ids
  std::map<int, size_t> mc_off;             // lgMc -> table offset
  std::map<int, McTabs> mc_tab;
  std::vector<size_t> sig_off;
  size_t off_desc = 0, off_sstats = 0, off_order = 0, off_mjobs = 0, off_msum = 0;
  // length classes run as tiled passes: partial slots [kind][signal][tile] per class
  std::map<int, size_t> tpart_off;
  std::map<int, int> tpart_tiles;
  // multi-dimensional groups
  std::vector<std::vector<int>> groups;
  std::vector<Plan> gplans;
  std::vector<size_t> goff;
  size_t bytes = 0;
};

int32_t batch_plan(int32_t dt, int32_t count, const ffcz_instance* inst, int32_t max_iter, BatchPlan& bp) {
  bp = BatchPlan();
  bp.dt = dt;
  if (dt != FFCZ_F32 && dt != FFCZ_F64) return fail(FFCZ_E_INVALID, "dtype must be FFCZ_F32 or FFCZ_F64");
  if (count < 0 || (count > 0 && !inst)) return fail(FFCZ_E_INVALID, "bad instance array");
  std::map<std::vector<int64_t>, int> gkey;
  for (int i = 0; i < count; ++i) {
    const ffcz_instance& in = inst[i];
    if (in.ndim < 1 || in.ndim > 3) return fail(FFCZ_E_SHAPE, "instance ndim must be 1..3");
    int64_t sq[3];
    for (int d = 0; d < in.ndim; ++d)
      if (in.shape[d] < 1) return fail(FFCZ_E_SHAPE, "every extent must be >= 1");
    const int nd = squeeze(in.ndim, in.shape, sq);
    if (nd <= 1) {
      const int64_t L = nd == 0 ? 1 : sq[0];
      if (L > (int64_t)1 << 19) return fail(FFCZ_E_SHAPE, "1D lengths must be at most 2^19");
      bp.sig_ids.push_back(i);
      continue;
    }
    std::vector<int64_t> key(sq, sq + nd);
    if (nd == 3) key.push_back(i);  // 3D instances run one at a time
    auto it = gkey.find(key);
    if (it == gkey.end()) {
      gkey[key] = (int)bp.groups.size();
      bp.groups.push_back({i});
    } else {
      bp.groups[it->second].push_back(i);
    }
  }
  size_t off = 0;
  for (auto& g : bp.groups) {
    Plan p;
    const ffcz_instance& in = inst[g[0]];
    int32_t r = make_plan(dt, in.ndim, in.shape, max_iter, (int64_t)g.size(), p);
    if (r != FFCZ_OK) return r;
    bp.gplans.push_back(p);
    bp.goff.push_back(off);
    off = align_up(off + p.bytes, 256);
  }
  const int ns = (int)bp.sig_ids.size();
  for (int k = 0; k < ns; ++k) {
    int64_t sq[3];
    const ffcz_instance& in = inst[bp.sig_ids[k]];
    const int nd = squeeze(in.ndim, in.shape, sq);
    SigPlan sp = sig_plan(dt, nd == 0 ? 1 : sq[0]);
    bp.sigs.push_back(sp);
    bp.by_mc[sp.lgMc].push_back(k);
    bp.sig_off.push_back(off);
    off = align_up(off + sp.bytes, 256);
  }
  for (auto& kv : bp.by_mc) {
    McTabs t = mc_tabs(dt, kv.first);
    bp.mc_tab[kv.first] = t;
    bp.mc_off[kv.first] = off;
    off = align_up(off + t.bytes, 256);
  }
  for (auto& kv : bp.by_mc) {
    if (kv.first < kSigTiledMinLg) continue;  // partial slots for every class that may run tiled
    int nct = 0, nrt = 0;
    sig_tiles(kv.first, &nct, &nrt);
    const int pt = std::max(nct, nrt);
    bp.tpart_off[kv.first] = off;
    bp.tpart_tiles[kv.first] = pt;
    off = align_up(off + sizeof(unsigned long long) * SP_KINDS * kv.second.size() * (size_t)pt, 256);
  }
  // margin jobs (x pointer, length, bound), descriptors and block order: one upload
  bp.off_mjobs = off;
  off = align_up(off + sizeof(MarginJob) * (size_t)std::max(count, 1), 256);
  bp.off_desc = off;
  off = align_up(off + sizeof(SigDesc) * (size_t)std::max(ns, 1), 256);
  bp.off_order = off;
  off = align_up(off + sizeof(int32_t) * (size_t)std::max(ns, 1), 256);
  bp.off_sstats = off;
  off = align_up(off + sizeof(SigStats) * (size_t)std::max(ns, 1), 256);
  bp.off_msum = off;  // margin partial sums (kUlpSlots per member), then the members' mu
  off = align_up(off + sizeof(double) * (size_t)(kUlpSlots + 1) * (size_t)std::max(count, 1), 256);
  bp.bytes = off;
  return FFCZ_OK;
}

// Tiled loop control, one block per signal slot of a length class: sum the
// check's partial counts (and the spatial-clip counts of the pass that made the
// checked iterate), record them, and decide whether the signal's loop ends.
__global__ void __launch_bounds__(256) sig_ctl_kernel(const SigDesc* sig, SigStats* stats, const int32_t* order,
                                                       const unsigned long long* part, int32_t nsig, int32_t ptiles,
                                                       int32_t nct, int32_t nrt, int32_t max_iter, int32_t fixed,
                                                       Post post) {
  __shared__ unsigned long long red[3][4];
  const int slot = blockIdx.x;
  if (slot >= nsig) return;
  const int sid = order[slot];
  SigStats* so = stats + sid;
  if (*(volatile int32_t*)&so->done) return;
  const int nck = sig[sid].blue ? nct : nrt;  // tiles of the pass that counted violations
  const int k = so->rounds;
  auto at = [&](int kind, int tl) { return part[((int64_t)kind * nsig + slot) * ptiles + tl]; };
  unsigned long long v = 0, z = 0, nf = 0;
  for (int i = threadIdx.x; i < nck; i += blockDim.x) v += at(SP_VIOL, i);
  for (int i = threadIdx.x; i < nct; i += blockDim.x) {
    z += at(SP_SCLIP, i);
    if (k == 0) nf += at(SP_NONFIN, i);
  }
  v = wave_sum_u64(v);
  z = wave_sum_u64(z);
  nf = wave_sum_u64(nf);
  if ((threadIdx.x & 63) == 0) {
    red[0][threadIdx.x >> 6] = v;
    red[1][threadIdx.x >> 6] = z;
    red[2][threadIdx.x >> 6] = nf;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long V = 0, Z = 0, NF = 0;
    for (int w = 0; w < (int)(blockDim.x + 63) / 64; ++w) {
      V += red[0][w];
      Z += red[1][w];
      NF += red[2][w];
    }
    if (k == 0) {
      so->s_guard = Z;
      so->viol0 = V;
    } else {
      so->s_clipped += Z;
    }
    so->violf = V;
    int stop = 0;
    if (k == 0 && NF) {
      so->nonfinite = NF;
      so->nonfinite_stop = 1;
      so->converged = 0;
      stop = 1;
    } else if (!fixed && V == 0) {
      so->converged = 1;
      stop = 1;
    } else if (k >= max_iter) {
      so->converged = (V == 0) ? 1 : 0;
      stop = 1;
    }
    if (stop) so->done = 1;
    else so->rounds = k + 1;
    post_check(post, slot, k + 1, stop);
  }
}

// Tiled verification totals, one block per signal slot.
__global__ void __launch_bounds__(256) sig_vstats_kernel(const SigDesc* sig, SigStats* stats, const int32_t* order,
                                                          const unsigned long long* part, int32_t nsig, int32_t ptiles,
                                                          int32_t nct, int32_t nrt) {
  __shared__ unsigned long long red[3][4];
  const int slot = blockIdx.x;
  if (slot >= nsig) return;
  const int sid = order[slot];
  SigStats* so = stats + sid;
  const int nv = sig[sid].blue ? nct : nrt;
  auto at = [&](int kind, int tl) { return part[((int64_t)kind * nsig + slot) * ptiles + tl]; };
  unsigned long long mf = 0, ms = 0, c = 0;  // maxima of non-negative doubles compare as their bits
  for (int i = threadIdx.x; i < nv; i += blockDim.x) {
    const unsigned long long b = at(SP_VMAXF, i);
    mf = mf > b ? mf : b;
    c += at(SP_VCNT, i);
  }
  for (int i = threadIdx.x; i < nct; i += blockDim.x) {
    const unsigned long long b = at(SP_VMAXS, i);
    ms = ms > b ? ms : b;
  }
  for (int off = 32; off > 0; off >>= 1) {
    const unsigned long long o1 = __shfl_xor(mf, off, 64), o2 = __shfl_xor(ms, off, 64);
    mf = mf > o1 ? mf : o1;
    ms = ms > o2 ? ms : o2;
    c += __shfl_xor(c, off, 64);
  }
  if ((threadIdx.x & 63) == 0) {
    red[0][threadIdx.x >> 6] = mf;
    red[1][threadIdx.x >> 6] = ms;
    red[2][threadIdx.x >> 6] = c;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long F = 0, S = 0, C = 0;
    for (int w = 0; w < (int)(blockDim.x + 63) / 64; ++w) {
      F = F > red[0][w] ? F : red[0][w];
      S = S > red[1][w] ? S : red[1][w];
      C += red[2][w];
    }
    so->max_spectral = __longlong_as_double((long long)F);
    so->max_spatial = __longlong_as_double((long long)S);
    so->spectral_viol = C;
  }
}

template <typename T>
hipError_t sig_launch(int dt, int mode, int lgMc, const BatchPlan& bp, char* ws, const int32_t* order,
                      int nsig, int32_t max_iter, int32_t fixed, hipStream_t s) {
  const McTabs& t = bp.mc_tab.at(lgMc);
  char* tb = ws + bp.mc_off.at(lgMc);
  const bool d64 = sig_mode_fp64(mode, dt);
  SigArgs<T> a;
  memset(&a, 0, sizeof(a));
  a.sig = (const SigDesc*)(ws + bp.off_desc);
  a.stats = (SigStats*)(ws + bp.off_sstats);
  a.order = order;
  a.nsig = nsig;
  a.max_iter = max_iter;
  a.fixed = fixed;
  a.tab.tw4 = (const cx<T>*)(tb + (d64 ? t.tw4_64 : t.tw4));
  a.tab.tw4r = (const cx<T>*)(tb + (d64 ? t.tw4r_64 : t.tw4r));
  a.tab.twa = (const cx<T>*)(tb + (d64 ? t.twa_64 : t.twa));
  a.tab.twb = (const cx<T>*)(tb + (d64 ? t.twb_64 : t.twb));
  auto it = bp.tpart_off.find(lgMc);
  if (it != bp.tpart_off.end()) {
    a.part = (unsigned long long*)(ws + it->second);
    a.ptiles = bp.tpart_tiles.at(lgMc);
  }
  return launch_sig(dt, mode, lgMc, &a, nsig, s);
}

// Margin jobs of every member, and descriptors (bounds, thresholds, buffer addresses) and block
// order of the 1D members, uploaded together; first[lg] is a class's first slot in the order.
// Without mus the descriptors' thresholds are left to margin_kernel.
int32_t sig_stage(const BatchPlan& bp, int32_t count, const ffcz_instance* inst, const double* mus, char* ws,
                  hipStream_t s, HostBuf& hsig, std::map<int, int>& first) {
  const int ns = (int)bp.sig_ids.size();
  // own staging buffer: the grouped members reuse g_host_init while this copy may be in flight
  const size_t bytes = bp.off_order + sizeof(int32_t) * (size_t)ns - bp.off_mjobs;
  HIPCHK(hsig.reserve(bytes));
  char* const h = (char*)hsig.p;
  MarginJob* hj = (MarginJob*)h;
  SigDesc* hd = (SigDesc*)(h + (bp.off_desc - bp.off_mjobs));
  int32_t* ho = (int32_t*)(h + (bp.off_order - bp.off_mjobs));
  for (int i = 0; i < count; ++i) {
    int64_t N = 1;
    for (int d = 0; d < inst[i].ndim; ++d) N *= inst[i].shape[d];
    hj[i] = MarginJob{(const float*)inst[i].x_orig, N, inst[i].delta_f, 0};
  }
  for (int k = 0; k < ns; ++k) {
    const int id = bp.sig_ids[k];
    const ffcz_instance& in = inst[id];
    const SigPlan& sp = bp.sigs[k];
    char* b = ws + bp.sig_off[k];
    hj[id].sig = k + 1;
    SigDesc d;
    memset(&d, 0, sizeof(d));
    d.x = in.x_orig;
    d.xb = in.x_base;
    d.y = in.x_out;
    d.L = sp.L;
    d.blue = sp.blue;
    d.E = in.eps_s;
    d.Delta = in.delta_f;
    if (mus) {
      d.Ep = in.eps_s * (1.0 - mus[id]);
      spectral_thresholds(bp.dt, in.delta_f, mus[id], &d.Dc, &d.Dp);
    }
    d.conv = b + sp.conv64;
    d.conv64 = b + sp.conv64;
    if (sp.blue) {
      d.btab = b + sp.btab;
      d.btab64 = b + sp.btab64;
      d.btabi = b + sp.btabi;
      d.chirp = b + sp.chirp;
      d.chirp64 = b + sp.chirp64;
    }
    d.eps = b + sp.eps;
    hd[k] = d;
  }
  // block order per convolution length: larger signals first
  int pos = 0;
  first.clear();
  for (auto& kv : bp.by_mc) {
    std::vector<int> ids = kv.second;
    std::sort(ids.begin(), ids.end(), [&](int a, int b) { return bp.sigs[a].L > bp.sigs[b].L; });
    first[kv.first] = pos;
    for (int id : ids) ho[pos++] = id;
  }
  HIPCHK(hipMemcpyAsync(ws + bp.off_mjobs, h, bytes, hipMemcpyHostToDevice, s));
  return FFCZ_OK;
}

// The four-step tables of every length class, and cleared loop states (one launch).
int32_t sig_tables(const BatchPlan& bp, char* ws, hipStream_t s) {
  if (bp.sig_ids.empty()) return FFCZ_OK;
  TabClasses J;
  memset(&J, 0, sizeof(J));
  int32_t nb = 0;
  for (auto& kv : bp.by_mc) {
    const int lg = kv.first, MA = sig_ma(lg), MB = (1 << lg) / MA;
    if (J.n >= 20) return fail(FFCZ_E_SHAPE, "too many 1D length classes");
    TabClass& c = J.c[J.n++];
    c.base = ws + bp.mc_off.at(lg);
    c.t = bp.mc_tab.at(lg);
    c.lgMc = lg;
    c.MA = MA;
    c.RR = sig_rows_per_tile(0, lg);
    c.first = nb;
    const int64_t n = ((int64_t)1 << lg) + host_twsize(MA, pick_E(MA)) + host_twsize(MB, pick_E(MB));
    nb += (int32_t)((n + 255) / 256);
  }
  J.dbl = bp.dt == FFCZ_F64 ? 1 : 0;
  J.zero = (unsigned long long*)(ws + bp.off_sstats);
  J.nzero = (int64_t)(bp.sig_ids.size() * sizeof(SigStats) / 8);
  J.zfirst = nb;
  nb += (int32_t)((J.nzero + 255) / 256);
  hipLaunchKernelGGL(sig_tables_kernel, dim3((unsigned)nb), dim3(256), 0, s, J);
  HIPCHK(hipGetLastError());
  return FFCZ_OK;
}

// One-block or tiled for a length class.  A threshold given in the options decides alone;
// otherwise classes below 2^kSigTiledMinLg run one block per signal, classes above 2^16 run
// tiled, and the ones between take the tuner's decision for (architecture, data type, work
// length, power-of-two bucket of the class's signal count, kinds of length): variant 0 is the
// default rule (tiled from 2^14), variant 1 the other form.  The key also names what was compared:
// the form of variant 0, whether the one-block loop is resident, and the revision of the two forms'
// kernels, to be raised with any change of either; an entry of another comparison is not found,
// and the class is timed again.
constexpr int kSigTuneMaxLg = 16;
constexpr int kSigFormRev = 2;
bool sig_default_tiled(int lg) { return lg >= 14; }
bool sig_resident(const ffcz_options& o, int dt, int lg) { return o.resident_1d != 0 && sig_res_fits(dt, lg); }
std::string sig_tune_key(const BatchPlan& bp, const ffcz_options& o, int lg) {
  const std::vector<int>& ids = bp.by_mc.at(lg);
  int n = 1;
  while (n < (int)ids.size()) n <<= 1;
  bool blue = false, p2 = false;
  for (int k : ids) (bp.sigs[k].blue ? blue : p2) = true;
  char buf[192];
  snprintf(buf, sizeof(buf), "%s %s sig lg=%d n<=%d kinds=%s%s 0=%s res=%d rev=%d", device_arch().c_str(),
           bp.dt == FFCZ_F32 ? "f32" : "f64", lg, n, blue ? "b" : "", p2 ? "p" : "",
           sig_default_tiled(lg) ? "tiled" : "block", sig_resident(o, bp.dt, lg) ? 1 : 0, kSigFormRev);
  return buf;
}

// The decision for class lg without timing (the table's entry, else the default rule).
int32_t sig_class_tiled(const BatchPlan& bp, const ffcz_options& o, int lg, hipStream_t s, bool* tiled) {
  if (o.tiled_1d_lg > 0) {
    *tiled = lg >= std::max(kSigTiledMinLg, (int)o.tiled_1d_lg);
    return FFCZ_OK;
  }
  if (lg < kSigTiledMinLg || lg > kSigTuneMaxLg) {
    *tiled = lg >= kSigTiledMinLg;
    return FFCZ_OK;
  }
  int v = 0;
  int32_t r = tune_pass(sig_tune_key(bp, o, lg), s, false, 0.9f, 2, [](int) { return hipSuccess; }, &v);
  if (r != FFCZ_OK) return r;
  *tiled = sig_default_tiled(lg) != (v == 1);
  return FFCZ_OK;
}

// A class's correction with a fixed number of rounds and no verification, one-block or tiled:
// the timing run of the tuner (writes the members' outputs, which the real run rewrites).
template <typename T>
hipError_t sig_trial(const BatchPlan& bp, char* ws, const int32_t* ord, int lg, bool tiled, bool resident,
                     int rounds, hipStream_t s) {
  const int nb = (int)bp.by_mc.at(lg).size();
  const int ns = (int)bp.sig_ids.size();
  auto go = [&](int mode) -> hipError_t {
    if (sig_mode_fp64(mode, bp.dt)) return sig_launch<double>(bp.dt, mode, lg, bp, ws, ord, nb, rounds, 1, s);
    return sig_launch<T>(bp.dt, mode, lg, bp, ws, ord, nb, rounds, 1, s);
  };
  hipLaunchKernelGGL(zero_u64_kernel, dim3((unsigned)((ns * sizeof(SigStats) / 8 + 255) / 256)), dim3(256), 0, s,
                     (unsigned long long*)(ws + bp.off_sstats), (int64_t)(ns * sizeof(SigStats) / 8));
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  bool blue = false, p2 = false;
  for (int k : bp.by_mc.at(lg)) (bp.sigs[k].blue ? blue : p2) = true;
  if (blue)
    for (int m : {(int)SIGT_CHIRP, (int)SIGT_BCOL, (int)SIGT_BROW})
      if ((e = go(m)) != hipSuccess) return e;
  if (!tiled) return go(resident ? SIG_RUNL : SIG_RUN);
  if ((e = go(SIGT_EPS0)) != hipSuccess) return e;
  if ((e = go(SIGT_CIN)) != hipSuccess) return e;
  int nct = 0, nrt = 0;
  sig_tiles(lg, &nct, &nrt);
  for (int r = 0; r <= rounds; ++r) {  // fixed rounds: the control stops the loop at the last check
    if (blue && (e = go(SIGT_RMUL)) != hipSuccess) return e;
    if (p2 && (e = go(SIGT_RCHECK)) != hipSuccess) return e;
    if (blue && (e = go(SIGT_CCHECK)) != hipSuccess) return e;
    hipLaunchKernelGGL(sig_ctl_kernel, dim3((unsigned)nb), dim3(256), 0, s, (const SigDesc*)(ws + bp.off_desc),
                       (SigStats*)(ws + bp.off_sstats), ord, (const unsigned long long*)(ws + bp.tpart_off.at(lg)),
                       (int32_t)nb, (int32_t)bp.tpart_tiles.at(lg), (int32_t)nct, (int32_t)nrt, (int32_t)rounds,
                       (int32_t)1, Post{nullptr, 0});
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (blue && (e = go(SIGT_RMULI)) != hipSuccess) return e;
    if ((e = go(SIGT_CSPAT)) != hipSuccess) return e;
  }
  return go(SIGT_Y);
}

// Time both forms of every class the tuner decides and has no entry for, on the call's own
// members (staged, with tables; three fixed rounds each, before the real run; nothing else runs
// meanwhile).
int32_t pretune_sigs(const BatchPlan& bp, const ffcz_options& o, char* ws, hipStream_t s,
                     const std::map<int, int>& first) {
  if (bp.sig_ids.empty() || o.tiled_1d_lg > 0) return FFCZ_OK;
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  HIPCHK(hipStreamIsCapturing(s, &cs));
  if (cs != hipStreamCaptureStatusNone) return FFCZ_OK;  // nothing is timed under capture
  bool ran = false;
  for (auto& kv : bp.by_mc) {
    const int lg = kv.first;
    if (lg < kSigTiledMinLg || lg > kSigTuneMaxLg) continue;
    const int32_t* ord = (const int32_t*)(ws + bp.off_order) + first.at(lg);
    const bool dflt = sig_default_tiled(lg);
    int v = 0;
    int32_t r = tune_pass(sig_tune_key(bp, o, lg), s, true, 0.9f, 2, [&](int var) {
      const bool tiled = dflt != (var == 1);
      ran = true;
      return bp.dt == FFCZ_F32 ? sig_trial<float>(bp, ws, ord, lg, tiled, sig_resident(o, bp.dt, lg), 3, s)
                               : sig_trial<double>(bp, ws, ord, lg, tiled, sig_resident(o, bp.dt, lg), 3, s);
    }, &v);
    if (r != FFCZ_OK) return r;
  }
  if (ran) {  // the trials used the loop states
    const int64_t n = (int64_t)(bp.sig_ids.size() * sizeof(SigStats) / 8);
    hipLaunchKernelGGL(zero_u64_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s,
                       (unsigned long long*)(ws + bp.off_sstats), n);
    HIPCHK(hipGetLastError());
  }
  return FFCZ_OK;
}

// Streams that independent length classes run on side by side: lane 0 is the stream that the
// work belongs to, the others are forked from it and joined into it.
struct SigLanes {
  int n = 1;
  hipStream_t q[3] = {nullptr, nullptr, nullptr};
};

// The 1D members of a batch in phases: begin (descriptors and tables are in place; the one-block
// classes on their own stream, the tiled classes' set-up), the tiled rounds (driven from here, or with
// the groups' rounds by the mixed-batch loop), end (the tiled classes' outputs
// and verification, then the one-block stream joined).  Every tiled round pass returns at entry
// once its signal's loop has ended.  A pass of one class is a small launch (10 to 40 us, mostly
// ramp and tail, few blocks for the shorter classes) and classes do not depend on each other, so
// they run in lanes: 128 EEG-like signals of 2^12 to 2^18 samples, one round of their five
// tiled classes one after another 450 us.
struct SigRun {
  const BatchPlan* bp = nullptr;
  int32_t max_iter = 0;
  ffcz_options o{};
  char* ws = nullptr;
  hipStream_t s = nullptr;       // set-up, tiled passes, end (lane 0)
  SigLanes lanes;                // the streams of set-up and end
  Streams* own = nullptr;        // the call's streams and events
  hipStream_t side = nullptr;    // one-block classes (joined into s at the end)
  hipEvent_t fork = nullptr, join = nullptr;
  std::map<int, int> first;      // class -> first slot in the block order
  std::vector<int> tiled;
  std::map<int, std::pair<bool, bool>> kinds;  // class -> (has Bluestein lengths, has power-of-two lengths)
  int fixed = 0, chunk = 4;
  bool side_used = false;

  const int32_t* order() const { return (const int32_t*)(ws + bp->off_order); }
  int nsig() const { return (int)bp->sig_ids.size(); }

  // a launch of one mode over every signal of class lg, in the mode's arithmetic, on st
  hipError_t go(int mode, int lg, hipStream_t st) const {
    const int nb = (int)bp->by_mc.at(lg).size();
    const int32_t* ord = order() + first.at(lg);
    if (sig_mode_fp64(mode, bp->dt)) return sig_launch<double>(bp->dt, mode, lg, *bp, ws, ord, nb, max_iter, fixed, st);
    return sig_launch<float>(bp->dt, mode, lg, *bp, ws, ord, nb, max_iter, fixed, st);
  }

  // the chirp and the spectra of its conjugate, tiled (Bluestein lengths)
  hipError_t setup_tables(int lg, hipStream_t st) const {
    hipError_t e = hipSuccess;
    if (kinds.at(lg).first)
      for (int m : {(int)SIGT_CHIRP, (int)SIGT_BCOL, (int)SIGT_BROW})
        if ((e = go(m, lg, st)) != hipSuccess) return e;
    return e;
  }

  // the FP64 verification of the members' outputs, tiled
  hipError_t verify_tiled(int lg, hipStream_t st) const {
    hipError_t e = go(SIGT_VCOL, lg, st);
    if (e != hipSuccess) return e;
    if ((e = go(SIGT_VROW, lg, st)) != hipSuccess) return e;
    if (kinds.at(lg).first && (e = go(SIGT_VCOL2, lg, st)) != hipSuccess) return e;
    int nct = 0, nrt = 0;
    sig_tiles(lg, &nct, &nrt);
    const int nb = (int)bp->by_mc.at(lg).size();
    hipLaunchKernelGGL(sig_vstats_kernel, dim3((unsigned)nb), dim3(256), 0, st, (const SigDesc*)(ws + bp->off_desc),
                       (SigStats*)(ws + bp->off_sstats), order() + first.at(lg),
                       (const unsigned long long*)(ws + bp->tpart_off.at(lg)), (int32_t)nb,
                       (int32_t)bp->tpart_tiles.at(lg), (int32_t)nct, (int32_t)nrt);
    return hipGetLastError();
  }

  int lanes_used(const SigLanes& L) const { return std::min<int>(L.n, (int)tiled.size()); }

  // f(class, stream) for every tiled class, classes spread over the lanes by their work (entries
  // of all signals; largest first onto the least loaded lane)
  template <typename F>
  hipError_t spread(const SigLanes& L, F&& f) const {
    const int n = lanes_used(L);
    std::vector<std::pair<int64_t, int>> w;
    for (int lg : tiled) w.push_back({(int64_t)bp->by_mc.at(lg).size() << lg, lg});
    std::sort(w.rbegin(), w.rend());
    hipError_t e = hipSuccess;
    int64_t load[3] = {0, 0, 0};
    for (size_t i = 0; i < w.size() && e == hipSuccess; ++i) {
      int k = 0;
      for (int j = 1; j < n; ++j)
        if (load[j] < load[k]) k = j;
      load[k] += w[i].first;
      e = f(w[i].second, L.q[k]);
    }
    return e;
  }

  // spread, with the other lanes forked from lane 0 before and joined into it after (also when a
  // launch failed)
  template <typename F>
  hipError_t across(const SigLanes& L, F&& f) const {
    const int n = lanes_used(L);
    hipError_t e = hipSuccess;
    if (n > 1) e = hipEventRecord(own->lfork, L.q[0]);
    for (int k = 1; k < n && e == hipSuccess; ++k) e = hipStreamWaitEvent(L.q[k], own->lfork, 0);
    if (e != hipSuccess) return e;
    e = spread(L, f);
    for (int k = 1; k < n; ++k) {
      hipError_t j = hipEventRecord(own->ljoin[k - 1], L.q[k]);
      if (j == hipSuccess) j = hipStreamWaitEvent(L.q[0], own->ljoin[k - 1], 0);
      if (e == hipSuccess) e = j;
    }
    return e;
  }

  int32_t begin(const BatchPlan& bp_, int32_t max_iter_, const ffcz_options& o_, char* ws_,
                const std::map<int, int>& first_, const SigLanes& lanes_, Streams& own_) {
    bp = &bp_;
    max_iter = max_iter_;
    o = o_;
    ws = ws_;
    first = first_;
    lanes = lanes_;
    s = lanes.q[0];
    own = &own_;
    side = own->side2;
    fork = own->fork2;
    join = own->join2;
    fixed = o.fixed_iterations ? 1 : 0;
    chunk = o.graph_chunk > 0 ? o.graph_chunk : 4;
    if (nsig() == 0) return FFCZ_OK;
    std::vector<int> oneblock;
    for (auto& kv : bp->by_mc) {
      const int lg = kv.first;
      bool is_tiled = false;
      int32_t tr = sig_class_tiled(*bp, o, lg, s, &is_tiled);
      if (tr != FFCZ_OK) return tr;
      bool b = false, p2 = false;
      for (int k : kv.second) (bp->sigs[k].blue ? b : p2) = true;
      kinds[lg] = {b, p2};
      (is_tiled ? tiled : oneblock).push_back(lg);
    }
    // the one-block classes run their whole correction on their own stream, beside the tiled
    // rounds (and, in a mixed batch, beside the grouped members: the set-up's end on s does
    // not wait for them); with no tiled classes there is nothing to run beside
    hipStream_t sb = s;
    if (!oneblock.empty() && side && !(tiled.empty() && bp->groups.empty())) {
      HIPCHK(hipEventRecord(fork, s));
      HIPCHK(hipStreamWaitEvent(side, fork, 0));
      sb = side;
      side_used = true;
    }
    for (int lg : oneblock) {
      // the loop in one launch; set-up and verification (FP64, in memory) tiled where those passes
      // exist: one block for them took 45 + 72 us of a single signal's call at Mc = 2^14
      const bool t = lg >= kSigTiledMinLg;
      if (t) HIPCHK(setup_tables(lg, sb));
      else HIPCHK(go(SIG_SETUP, lg, sb));
      HIPCHK(go(sig_resident(o, bp->dt, lg) ? SIG_RUNL : SIG_RUN, lg, sb));
      if (!o.verify_fp64) continue;
      if (t) HIPCHK(verify_tiled(lg, sb));
      else HIPCHK(go(SIG_VERIFY, lg, sb));
    }
    // tiled classes: set-up, eps0 and the first forward column pass
    HIPCHK(across(lanes, [&](int lg, hipStream_t st) {
      hipError_t e = setup_tables(lg, st);
      if (e != hipSuccess) return e;
      if ((e = go(SIGT_EPS0, lg, st)) != hipSuccess) return e;
      return go(SIGT_CIN, lg, st);
    }));
    return FFCZ_OK;
  }

  // one round of class lg on st, checks posted to post
  hipError_t round_of(int lg, hipStream_t st, const Post& post) const {
    const bool b = kinds.at(lg).first, p2 = kinds.at(lg).second;
    int nct = 0, nrt = 0;
    sig_tiles(lg, &nct, &nrt);
    const int nb = (int)bp->by_mc.at(lg).size();
    hipError_t e = hipSuccess;
    if (b && (e = go(SIGT_RMUL, lg, st)) != hipSuccess) return e;
    if (p2 && (e = go(SIGT_RCHECK, lg, st)) != hipSuccess) return e;
    if (b && (e = go(SIGT_CCHECK, lg, st)) != hipSuccess) return e;
    hipLaunchKernelGGL(sig_ctl_kernel, dim3((unsigned)nb), dim3(256), 0, st, (const SigDesc*)(ws + bp->off_desc),
                       (SigStats*)(ws + bp->off_sstats), order() + first.at(lg),
                       (const unsigned long long*)(ws + bp->tpart_off.at(lg)), (int32_t)nb,
                       (int32_t)bp->tpart_tiles.at(lg), (int32_t)nct, (int32_t)nrt, max_iter, (int32_t)fixed, post);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (b && (e = go(SIGT_RMULI, lg, st)) != hipSuccess) return e;
    return go(SIGT_CSPAT, lg, st);
  }

  // the rounds of every tiled class as tasks of drive(), checks posted from word w0 on; returns the
  // first word past them
  size_t tasks(std::vector<RoundTask>& out, size_t w0) {
    (void)spread(lanes, [&](int lg, hipStream_t st) {
      const size_t n = bp->by_mc.at(lg).size();
      const Post post = g_posts.at(w0);
      out.push_back(RoundTask{st, w0, n, [this, lg, st, post](int) { return round_of(lg, st, post); }});
      w0 += n;
      return hipSuccess;
    });
    return w0;
  }

  // one chunk of rounds of every tiled class
  hipError_t enqueue_chunk() const {
    return across(lanes, [&](int lg, hipStream_t st) {
      hipError_t e = hipSuccess;
      for (int r = 0; r < chunk && e == hipSuccess; ++r) e = round_of(lg, st, Post{nullptr, 0});
      return e;
    });
  }

  // whether every tiled signal's loop has ended, from a host copy of the signal states
  bool all_done(const SigStats* hs) const {
    for (int lg : tiled)
      for (int k : bp->by_mc.at(lg))
        if (!hs[k].done) return false;
    return true;
  }

  // the tiled rounds driven from here: round by round as checks are posted, or, on request, in
  // chunks with one poll of the done-flags per chunk
  int32_t loop(HostBuf& hstate) {
    if (tiled.empty()) return FFCZ_OK;
    const int ns = nsig();
    if (o.use_graph) {
      HIPCHK(g_posts.start((size_t)ns));
      std::vector<RoundTask> t;
      tasks(t, 0);
      return drive(t, max_iter);
    }
    HIPCHK(hstate.reserve(sizeof(SigStats) * ns));
    SigStats* hs = (SigStats*)hstate.p;
    for (int enq = 0;; enq += chunk) {
      HIPCHK(enqueue_chunk());
      HIPCHK(hipMemcpyAsync(hs, ws + bp->off_sstats, sizeof(SigStats) * ns, hipMemcpyDeviceToHost, s));
      HIPCHK(hipStreamSynchronize(s));
      if (all_done(hs)) break;
      if (enq > max_iter + 2 * chunk + 2) return fail(FFCZ_E_HIP, "tiled signals did not report completion");
    }
    return FFCZ_OK;
  }

  // the tiled classes' outputs and verification, then s waits for the one-block classes
  int32_t end() {
    HIPCHK(across(lanes, [&](int lg, hipStream_t st) {
      const hipError_t e = go(SIGT_Y, lg, st);
      return e != hipSuccess || !o.verify_fp64 ? e : verify_tiled(lg, st);
    }));
    lanes.n = 1;  // joined
    return rejoin();
  }

  // s waits for the other lanes and the one-block stream (also on early exits, so no launch
  // outlives the call)
  int32_t rejoin() {
    for (int k = 1; k < lanes.n && lanes.q[k]; ++k) {
      HIPCHK(hipEventRecord(own->ljoin[k - 1], lanes.q[k]));
      HIPCHK(hipStreamWaitEvent(s, own->ljoin[k - 1], 0));
    }
    lanes.n = 1;
    if (!side_used) return FFCZ_OK;
    side_used = false;
    HIPCHK(hipEventRecord(join, side));
    HIPCHK(hipStreamWaitEvent(s, join, 0));
    return FFCZ_OK;
  }
  ~SigRun() { (void)rejoin(); }
};

int32_t run_sigs(const BatchPlan& bp, int32_t max_iter, const ffcz_options& o, char* ws, hipStream_t s,
                 const std::map<int, int>& first, HostBuf& hstate) {
  if (bp.sig_ids.empty()) return FFCZ_OK;
  Streams* q = nullptr;
  HIPCHK(streams_of(s, &q));
  SigRun sr;
  int32_t r = sr.begin(bp, max_iter, o, ws, first, SigLanes{3, {s, q->lane1, q->side}}, *q);
  if (r != FFCZ_OK) return r;
  r = sr.loop(hstate);
  if (r != FFCZ_OK) return r;
  return sr.end();
}

// dmu: the members' margins on the device, where the host does not have them yet (else null).
int32_t collect_sigs(const BatchPlan& bp, const ffcz_instance* inst, std::vector<double>& mus, const double* dmu,
                     const ffcz_options& o, char* ws, hipStream_t s, ffcz_stats* stats, int32_t* status) {
  const int ns = (int)bp.sig_ids.size();
  if (ns == 0) return FFCZ_OK;
  HIPCHK(g_host_misc.reserve(sizeof(SigStats) * ns + sizeof(double) * mus.size()));
  SigStats* h = (SigStats*)g_host_misc.p;
  double* hmu = (double*)(h + ns);
  HIPCHK(hipMemcpyAsync(h, ws + bp.off_sstats, sizeof(SigStats) * ns, hipMemcpyDeviceToHost, s));
  if (dmu) HIPCHK(hipMemcpyAsync(hmu, dmu, sizeof(double) * mus.size(), hipMemcpyDeviceToHost, s));
  HIPCHK(hipStreamSynchronize(s));
  if (dmu) mus.assign(hmu, hmu + mus.size());
  for (int k = 0; k < ns; ++k) {
    const int id = bp.sig_ids[k];
    const SigStats& g = h[k];
    if (stats) {
      ffcz_stats& st = stats[id];
      memset(&st, 0, sizeof(st));
      st.rounds = g.rounds;
      st.converged = g.converged;
      st.f_viol_initial = (int64_t)g.viol0;
      st.f_viol_final = (int64_t)g.violf;
      st.s_clipped_total = (int64_t)g.s_clipped;
      st.s_guard = (int64_t)g.s_guard;
      st.nonfinite = (int64_t)g.nonfinite;
      st.max_spatial_err = o.verify_fp64 ? g.max_spatial : NAN;
      st.max_spectral_err = o.verify_fp64 ? g.max_spectral : NAN;
      st.spectral_viol = (int64_t)g.spectral_viol;
      st.margin_used = mus[id];
    }
    int32_t r = FFCZ_OK;
    if (g.nonfinite_stop) r = FFCZ_E_NONFINITE;
    else if (!g.converged && !o.fixed_iterations) r = FFCZ_NOT_CONVERGED;
    else if (o.verify_fp64 && (!(g.max_spatial <= inst[id].eps_s) || !(g.max_spectral <= inst[id].delta_f)))
      r = FFCZ_VERIFY_FAILED;
    status[id] = r;
  }
  return FFCZ_OK;
}

// Streaming copy: one 16-byte vector per lane, one block per 4 KiB (measured on
// MI355X as the fastest of the simple forms: more work per lane or a grid-stride
// loop keeps fewer requests in flight).
__global__ void __launch_bounds__(256) copy_kernel(uint4* __restrict__ dst, const uint4* __restrict__ src,
                                                   int64_t n16) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n16) dst[i] = src[i];
}

__global__ void copy_tail_kernel(unsigned char* __restrict__ dst, const unsigned char* __restrict__ src, int n) {
  if ((int)threadIdx.x < n) dst[threadIdx.x] = src[threadIdx.x];
}

// Copy with the access pattern of the strided-axis passes: block (f, tile) moves the
// 128-byte tile of the rows (f, i) for every i along the axis, 16 bytes per lane, 8 lanes
// per tile row and 32 rows per step.  Row (f, i) starts at f fixed_stride + i axis_stride.
__global__ void __launch_bounds__(256) copy_columns_kernel(char* __restrict__ dst, const char* __restrict__ src,
                                                           int64_t n_axis, int64_t axis_stride, int64_t fixed_stride,
                                                           int64_t row_bytes, int32_t tiles) {
  const int64_t b = blockIdx.x;
  const int64_t f = b / tiles;
  const int tile = (int)(b - f * tiles);
  const int64_t off = (int64_t)tile * 128 + (threadIdx.x & 7) * 16;
  if (off >= row_bytes) return;  // row_bytes is a multiple of 16; no barrier follows
  const int64_t base = f * fixed_stride + off;
#pragma unroll 4
  for (int64_t i = threadIdx.x >> 3; i < n_axis; i += 32) {
    const int64_t a = base + i * axis_stride;
    *reinterpret_cast<uint4*>(dst + a) = *reinterpret_cast<const uint4*>(src + a);
  }
}

// Makes the caller's stream wait for the side stream on every exit after the fork, so no
// 1D launch still writes the caller's buffers once the call has returned.
struct SideJoin {
  hipStream_t s = nullptr, s1 = nullptr;
  hipEvent_t join = nullptr;
  ~SideJoin() {
    if (s1 && s1 != s) {
      (void)hipEventRecord(join, s1);
      (void)hipStreamWaitEvent(s, join, 0);
    }
  }
};


// A batch of 1D and grouped members, driven from the calling thread.  Everything is tuned
// first, with nothing else running.  Then the 1D set-up runs on side streams (its one-block
// classes on one of their own, beside everything else) while the groups' set-up runs on the
// caller's stream; the rounds of every group and of every tiled 1D class advance on their own as
// their checks are posted; last, the groups' closing passes on the caller's stream and the tiled
// classes' outputs and verification on the side streams, joined before return.
template <typename T>
int32_t mixed_batch(const BatchPlan& bp, const ffcz_instance* inst, const std::vector<double>& mus,
                    int32_t max_iter, const ffcz_options& o, char* w, hipStream_t s, const std::map<int, int>& first,
                    ffcz_stats* stats, std::vector<int32_t>& status) {
  for (size_t g = 0; g < bp.groups.size(); ++g) {
    int32_t r = pretune_group<T>(bp.gplans[g], w + bp.goff[g], s);
    if (r != FFCZ_OK) return r;
  }
  int32_t r = pretune_sigs(bp, o, w, s, first);
  if (r != FFCZ_OK) return r;
  Streams* q = nullptr;
  HIPCHK(streams_of(s, &q));
  const hipStream_t s1 = q->side;
  HIPCHK(hipEventRecord(q->fork, s));
  HIPCHK(hipStreamWaitEvent(s1, q->fork, 0));
  SideJoin side;  // s waits for s1 on every exit from here
  side.s = s;
  side.s1 = s1;
  side.join = q->join;
  SigRun sr;      // declared after the join: its own stream joins s1 first
  r = sr.begin(bp, max_iter, o, w, first, SigLanes{2, {s1, q->lane1, nullptr}}, *q);
  if (r != FFCZ_OK) return r;
  // the groups' set-up on s; their instance and margin arrays live as long as the runs
  const size_t ng = bp.groups.size();
  std::vector<std::vector<ffcz_instance>> gis(ng);
  std::vector<std::vector<double>> gms(ng);
  std::vector<std::unique_ptr<GroupRun<T>>> gr;
  for (size_t g = 0; g < ng; ++g) {
    for (int id : bp.groups[g]) {
      gis[g].push_back(inst[id]);
      gms[g].push_back(mus[id]);
    }
    gr.emplace_back(new GroupRun<T>());
    r = gr.back()->begin(bp.gplans[g], gis[g].data(), gms[g].data(), max_iter, o, w + bp.goff[g], s, nullptr,
                         nullptr, nullptr);
    if (r != FFCZ_OK) return r;
  }
  if (o.use_graph || o.fixed_iterations) {
    // every group's and every tiled class's rounds side by side; fixed rounds end by their
    // control kernels too
    size_t words = bp.sig_ids.size(), w0 = 0;
    for (const Plan& gp : bp.gplans) words += (size_t)gp.B;
    HIPCHK(g_posts.start(words));
    std::vector<RoundTask> t;
    for (size_t g = 0; g < ng; ++g) {
      t.push_back(gr[g]->task(w0));
      w0 += (size_t)bp.gplans[g].B;
    }
    sr.tasks(t, w0);
    r = drive(t, max_iter);
    if (r != FFCZ_OK) return r;
  } else {
    // chunks of everything, with one poll of every group's states and the signal states per chunk
    size_t hbytes = sizeof(SigStats) * bp.sig_ids.size();
    std::vector<size_t> hoff(ng);
    for (size_t g = 0; g < ng; ++g) {
      hoff[g] = hbytes;
      hbytes += sizeof(DevState) * (size_t)bp.gplans[g].B;
    }
    HIPCHK(g_host_sigstate.reserve(hbytes));
    char* hb = (char*)g_host_sigstate.p;
    const int chunk = o.graph_chunk > 0 ? o.graph_chunk : 4;
    for (int enq = 0;; enq += chunk) {
      for (size_t g = 0; g < ng; ++g)
        for (int k = 0; k < chunk; ++k) HIPCHK(gr[g]->round(enq + k));
      HIPCHK(sr.enqueue_chunk());
      HIPCHK(hipMemcpyAsync(hb, w + bp.off_sstats, sizeof(SigStats) * bp.sig_ids.size(), hipMemcpyDeviceToHost, s1));
      for (size_t g = 0; g < ng; ++g)
        HIPCHK(hipMemcpyAsync(hb + hoff[g], gr[g]->c.st(), sizeof(DevState) * (size_t)bp.gplans[g].B,
                              hipMemcpyDeviceToHost, s));
      HIPCHK(hipStreamSynchronize(s1));
      HIPCHK(hipStreamSynchronize(s));
      bool all = sr.all_done((const SigStats*)hb);
      for (size_t g = 0; g < ng && all; ++g) {
        const DevState* hs = (const DevState*)(hb + hoff[g]);
        for (int64_t b = 0; b < bp.gplans[g].B; ++b) all = all && hs[b].done;
      }
      if (all) break;
      if (enq > max_iter + 2 * chunk + 2) return fail(FFCZ_E_HIP, "batch did not report completion");
    }
  }
  // the tiled classes' end on their lanes, the groups' ends on s
  r = sr.end();
  if (r != FFCZ_OK) return r;
  for (size_t g = 0; g < ng; ++g) {
    std::vector<int32_t> gs(gis[g].size(), FFCZ_OK);
    std::vector<ffcz_stats> gst(gis[g].size());
    r = gr[g]->end(gst.data(), gs.data());
    if (r != FFCZ_OK) return r;
    for (size_t k = 0; k < gis[g].size(); ++k) {
      status[bp.groups[g][k]] = gs[k];
      if (stats) stats[bp.groups[g][k]] = gst[k];
    }
  }
  return FFCZ_OK;
}

int32_t worst(const std::vector<int32_t>& st) {
  int32_t w = FFCZ_OK;
  for (int32_t v : st) {
    if (v < 0) return v;
    w = std::max(w, v);
  }
  return w;
}

// Checked arguments of a single-field call on the plan path.
struct SingleCall {
  Plan p;
  ffcz_options o;
  double mu = 0.0;
  ffcz_instance in;
};

int32_t single_setup(int32_t dtype, int32_t ndim, const int64_t* shape, const void* x, const void* xb, void* y,
                     double eps_s, double delta_f, int32_t max_iter, const ffcz_options* opts, SingleCall& sc) {
  int32_t r = make_plan(dtype, ndim, shape, max_iter, 1, sc.p);
  if (r != FFCZ_OK) return r;
  if (!x || !xb || !y) return fail(FFCZ_E_INVALID, "null data pointer");
  if (x == xb || x == y) return fail(FFCZ_E_INVALID, "x_orig must not alias x_base or x_out");
  if (!std::isfinite(eps_s) || eps_s < 0) return fail(FFCZ_E_INVALID, "eps_s must be finite and >= 0");
  if (!std::isfinite(delta_f) || delta_f < 0) return fail(FFCZ_E_INVALID, "delta_f must be finite and >= 0");
  if (((uintptr_t)x & 15) || ((uintptr_t)xb & 15) || ((uintptr_t)y & 15))
    return fail(FFCZ_E_WORKSPACE, "data pointers must be 16-byte aligned");
  if (opts) sc.o = *opts;
  else ffcz_default_options(&sc.o);
  if (sc.o.masks_out && sc.p.dt == FFCZ_F64 && col_block_cols(1, sc.p.Lx, 0) < 8)
    return fail(FFCZ_E_SHAPE, "mask recording needs at least 8 columns per block");
  // no margin given: FP64 takes 2^-16, FP32 derives mu from x on the device (no host round trip)
  sc.mu = sc.o.margin_rel > 0.0 ? sc.o.margin_rel : (dtype == FFCZ_F64 ? std::ldexp(1.0, -16) : 0.0);
  if (!(sc.mu < 1.0)) return fail(FFCZ_E_INVALID, "margin_rel must be in [0, 1)");
  memset(&sc.in, 0, sizeof(sc.in));
  sc.in.ndim = ndim;
  for (int i = 0; i < ndim; ++i) sc.in.shape[i] = shape[i];
  sc.in.x_orig = x;
  sc.in.x_base = xb;
  sc.in.x_out = y;
  sc.in.eps_s = eps_s;
  sc.in.delta_f = delta_f;
  return FFCZ_OK;
}

// host_state: null for the ordinary call; else the no-allocation form (see correct_group).
int32_t single_run(SingleCall& sc, char* ws, hipStream_t s, ffcz_stats* stats, DevState* host_state) {
  const double* mus = sc.mu > 0.0 ? &sc.mu : nullptr;
  int32_t status = FFCZ_OK;
  const int32_t r =
      sc.p.dt == FFCZ_F32
          ? correct_group<float>(sc.p, &sc.in, mus, sc.p.max_iter, sc.o, ws, s, stats, &status, host_state)
          : correct_group<double>(sc.p, &sc.in, mus, sc.p.max_iter, sc.o, ws, s, stats, &status, host_state);
  if (r != FFCZ_OK) return r;
  if (stats) stats->status = status;
  if (status == FFCZ_E_NONFINITE) return fail(FFCZ_E_NONFINITE, "x or x_hat holds NaN or Inf");
  if (status == FFCZ_VERIFY_FAILED) g_err = "FP64 re-verification failed";
  return status;
}

// Flags and codes of both sets (status and totals written on the device).
template <typename T>
hipError_t code_sets(const EditJob<T>& a, const EditJob<T>& b, unsigned* status, hipStream_t s) {
  const unsigned nb = (unsigned)(a.nb + b.nb);
  if (nb) hipLaunchKernelGGL(edit_count_kernel<T>, dim3(nb), dim3(64 * kEditWaves), 0, s, a, b);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(edit_scan_kernel, dim3(2), dim3(1024), 0, s, ScanJob{a.off, a.nb, a.total},
                     ScanJob{b.off, b.nb, b.total}, status);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (nb) hipLaunchKernelGGL(edit_write_kernel<T>, dim3(nb), dim3(64 * kEditWaves), 0, s, a, b, status);
  return hipGetLastError();
}

// The inverse for the decoder: dense dequantised edits from flags and codes.
template <typename TO>
hipError_t expand_sets(const EditJob<TO>& a, const EditJob<TO>& b, unsigned* status, hipStream_t s) {
  const unsigned nb = (unsigned)(a.nb + b.nb);
  if (nb) hipLaunchKernelGGL(flag_count_kernel<TO>, dim3((nb + 3) / 4), dim3(256), 0, s, a, b);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(edit_scan_kernel, dim3(2), dim3(1024), 0, s, ScanJob{a.off, a.nb, a.total},
                     ScanJob{b.off, b.nb, b.total}, status);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (nb) hipLaunchKernelGGL(edit_expand_kernel<TO>, dim3(nb), dim3(64 * kEditWaves), 0, s, a, b, status);
  return hipGetLastError();
}

template <typename T>
EditSet<T> spatial_set(void* base, int64_t n) {
  EditSet<T> e;
  memset(&e, 0, sizeof(e));
  e.val = (T*)base;
  e.ncoord = n;
  return e;
}
template <typename T>
EditSet<T> freq_set(const Plan& p, void* spec) {
  EditSet<T> e;
  memset(&e, 0, sizeof(e));
  e.val = (T*)spec;
  e.ncoord = 2 * p.nrows * p.ncols;
  e.freq = 1;
  e.ncols = (int32_t)p.ncols;
  e.pitch = p.pitch;
  e.plane = p.plane;
  e.lg_rpp = p.lg_rpp;
  e.inv = 1.0 / (double)p.ncols;
  return e;
}

// Encoder after the loop: code both sets, export the accumulators when asked, and read
// back the code counts and the status word.
template <typename T>
int32_t code_edits(const Plan& p, const EditLayout& L, char* ws, void* sflags, int32_t* scodes, void* fflags,
                   int32_t* fcodes, double step_s, double step_f, void* sexp, void* fexp, hipStream_t s,
                   int64_t* nnz_s, int64_t* nnz_f) {
  unsigned long long* tot = (unsigned long long*)(ws + L.off_tot);
  unsigned* status = (unsigned*)(tot + 2);
  const EditSet<T> ss = spatial_set<T>(ws + L.off_S, L.ncs);
  const EditSet<T> fs = freq_set<T>(p, ws + L.off_F);
  HIPCHK(code_sets<T>({ss, L.nbs, (unsigned long long*)(ws + L.off_offs), tot, (uint8_t*)sflags, scodes, 0, step_s},
                      {fs, L.nbf, (unsigned long long*)(ws + L.off_offf), tot + 1, (uint8_t*)fflags, fcodes, 0, step_f},
                      status, s));
  if (sexp && L.ncs) {
    hipLaunchKernelGGL(edit_export_kernel<T>, dim3((unsigned)((L.ncs + 255) / 256)), dim3(256), 0, s, ss, (T*)sexp);
    HIPCHK(hipGetLastError());
  }
  if (fexp && L.ncf) {
    hipLaunchKernelGGL(edit_export_kernel<T>, dim3((unsigned)((L.ncf + 255) / 256)), dim3(256), 0, s, fs, (T*)fexp);
    HIPCHK(hipGetLastError());
  }
  unsigned long long h[3];
  HIPCHK(hipMemcpyAsync(h, tot, sizeof(h), hipMemcpyDeviceToHost, s));
  HIPCHK(hipStreamSynchronize(s));
  *nnz_s = (int64_t)h[0];
  *nnz_f = (int64_t)h[1];
  if ((unsigned)h[2] & kEditCodeRange)
    return fail(FFCZ_E_INVALID, "an edit's code falls outside int32 (fewer code bits m, or a zero bound with edits)");
  return FFCZ_OK;
}

// Decoder: y = x_hat + s + IFFT(f) from flags and codes (Sec. IV-B, applying edits).
template <typename T>
int32_t decode_impl(const Plan& p, const EditLayout& L, char* ws, const void* xb, const void* sflags,
                    const int32_t* scodes, int64_t nnz_s, const void* fflags, const int32_t* fcodes, int64_t nnz_f,
                    double step_s, double step_f, void* y, hipStream_t s) {
  Ctx c{&p, ws, s};
  StateInit si;
  memset(&si, 0, sizeof(si));
  si.inv_n = 1.0 / (double)p.N;
  si.px = y;  // the expanded spatial edits, read back by the closing pass
  si.pxb = xb;
  si.py = y;
  unsigned long long* tot = (unsigned long long*)(ws + L.off_tot);
  HIPCHK(run_setup(c, nullptr, si, nullptr, 0));
  unsigned* status = (unsigned*)(tot + 2);
  // spatial edits straight into y (the field's dtype), frequency edits into Z
  HIPCHK(expand_sets<T>({spatial_set<T>(y, L.ncs), L.nbs, (unsigned long long*)(ws + L.off_offs), tot,
                         (uint8_t*)sflags, (int32_t*)scodes, nnz_s, step_s},
                        {freq_set<T>(p, c.Z()), L.nbf, (unsigned long long*)(ws + L.off_offf), tot + 1,
                         (uint8_t*)fflags, (int32_t*)fcodes, nnz_f, step_f},
                        status, s));
  // inverse transforms: x, then y (3D), then the last-axis C2R with 1/N and the sum
  const char* twb = (const char*)c.twT();
  HIPCHK(run_col<T>(p.dt, COL_INV_NS, 0, geom_x(p, p.pitch, p.plane), p, c.Z(), c.Z(), twb + sizeof(cx<T>) * p.twx,
                    c.st(), nullptr, nullptr, s));
  if (p.nd == 3)
    HIPCHK(run_col<T>(p.dt, COL_INV_NS, 0, geom_y(p, p.pitch, p.plane), p, c.Z(), c.Z(),
                      twb + sizeof(cx<T>) * p.twy, c.st(), nullptr, nullptr, s));
  const hipError_t de = run_row<T, T>(p.dt, p.dt, ROW_DECODE, 0, p, p.pitch, p.plane, c.Z(), nullptr,
                                      twb + sizeof(cx<T>) * p.twz, c.st(), nullptr, nullptr, s);
  HIPCHK(de);
  unsigned long long h[3];
  HIPCHK(hipMemcpyAsync(h, tot, sizeof(h), hipMemcpyDeviceToHost, s));
  HIPCHK(hipStreamSynchronize(s));
  if ((unsigned)h[2] & kEditFlagCount)
    return fail(FFCZ_E_INVALID, "the set flags and the code counts given disagree (spatial " +
                                    std::to_string(h[0]) + " vs " + std::to_string(nnz_s) + ", frequency " +
                                    std::to_string(h[1]) + " vs " + std::to_string(nnz_f) + ")");
  return FFCZ_OK;
}

// Pointwise spectral bound that keeps every shell of the power spectrum of x within rho:
// FP64 spectrum of x on the verification passes (their last-axis pass forms y - x; here y = x
// and no x is given, read as zero), shell sums, shell bounds, then the bound of every entry.
template <typename T>
int32_t power_bounds_impl(const Plan& p, const BoundsLayout& L, char* ws, const void* x, double rho, int disk,
                          void* out, hipStream_t s) {
  Ctx c{&p, ws, s};
  StateInit si;
  memset(&si, 0, sizeof(si));
  si.inv_n = 1.0 / (double)p.N;
  si.py = const_cast<void*>(x);
  HIPCHK(run_setup(c, nullptr, si, nullptr, 0));
  const char* tb = (const char*)c.tw64();
  void* W = c.W();
  const hipError_t ez = run_row<double, T>(1, p.dt, ROW_VERIFY, kVerifyRowPlan, p, p.pitch64, p.plane64, nullptr, W,
                                           tb + 16 * p.twz8, c.st(), c.part(Ctx::PVZ), nullptr, s);
  HIPCHK(ez);
  if (p.nd == 3)
    HIPCHK(run_col<double>(1, COL_FWD_NS, 0, geom_y(p, p.pitch64, p.plane64), p, W, W, tb + 16 * p.twy, c.st(),
                           nullptr, nullptr, s));
  if (p.nd >= 2)
    HIPCHK(run_col<double>(1, COL_FWD_NS, 0, geom_x(p, p.pitch64, p.plane64), p, W, W, tb + 16 * p.twx, c.st(),
                           nullptr, nullptr, s));
  const SpecGeom g64{p.nrows, (int32_t)p.ncols, p.lg_rpp, p.pitch64, p.plane64};
  const int n0 = p.nd >= 2 ? (int)p.n[0] : 1, lg1 = p.nd == 3 ? ilog2c((int)p.n[1]) : 0, nl = (int)p.n[p.nd - 1];
  double* part = (double*)(ws + L.off_shell);
  double* bins = (double*)(ws + L.off_bins);
  hipLaunchKernelGGL(shell_part_kernel, dim3((unsigned)L.nsb), dim3(kShellLanes), 0, s, (const cx<double>*)W, g64, p.nd,
                     n0, lg1, nl, L.nb, part);
  HIPCHK(hipGetLastError());
  hipLaunchKernelGGL(shell_bound_kernel, dim3((unsigned)((L.nb + 15) / 16)), dim3(1024), 0, s,
                     (const double*)part, L.nsb, L.nb, rho, disk, bins);
  HIPCHK(hipGetLastError());
  const int64_t M = p.nrows * p.ncols;
  hipLaunchKernelGGL(shell_scatter_kernel<T>, dim3((unsigned)std::min<int64_t>(4096, (M + 255) / 256)), dim3(256), 0,
                     s, (const double*)bins, p.nrows, (int32_t)p.ncols, p.nd, n0, lg1, (T*)out);
  HIPCHK(hipGetLastError());
  return FFCZ_OK;
}

// ---------------------------------------------------------------------------
// Huffman code construction (host side of LosslesslyCompressEdits).  The tree merges the two
// lightest nodes, ties going to the node created first (leaves in symbol order, then merged
// nodes in turn), so the code lengths depend on the frequency table alone; codes longer than
// kHuffMaxLen bits make every non-zero count (count + 1) / 2 and the tree is rebuilt.

constexpr int kHuffMaxLen = 32;
constexpr int64_t kHuffMaxAlpha = int64_t(1) << 24;

// The merges in O(n) after a sort: leaves sorted by (count, symbol), merged nodes appended to a
// second queue in creation order.  Merged weights never decrease, so both queues stay ordered
// by (weight, id) and the lighter front is the node a heap ordered by (weight, id) would pop
// (on equal weights the leaf, whose id is the smaller).
std::vector<uint8_t> huff_tree_lengths(const std::vector<unsigned long long>& c) {
  std::vector<uint8_t> len(c.size(), 0);
  std::vector<int64_t> present;
  std::vector<unsigned long long> w;  // leaf weights, leaf id = position in present
  for (size_t i = 0; i < c.size(); ++i)
    if (c[i]) {
      present.push_back((int64_t)i);
      w.push_back(c[i]);
    }
  const int64_t nl = (int64_t)present.size();
  if (nl == 0) return len;
  if (nl == 1) {
    len[present[0]] = 1;
    return len;
  }
  // sort the leaf ids by (weight, id): least significant digit radix sort on 11-bit digits
  // (stable, so equal weights keep id order)
  std::vector<int64_t> leaf(nl), tmp(nl);
  for (int64_t i = 0; i < nl; ++i) leaf[i] = i;
  unsigned long long wmax = 0;
  for (int64_t i = 0; i < nl; ++i) wmax = std::max(wmax, w[i]);
  for (int sh = 0; sh < 64 && (wmax >> sh) != 0; sh += 11) {
    std::vector<int64_t> bucket(2049, 0);
    for (int64_t i = 0; i < nl; ++i) bucket[((w[leaf[i]] >> sh) & 2047) + 1]++;
    for (int d = 0; d < 2048; ++d) bucket[d + 1] += bucket[d];
    for (int64_t i = 0; i < nl; ++i) tmp[bucket[(w[leaf[i]] >> sh) & 2047]++] = leaf[i];
    leaf.swap(tmp);
  }
  std::vector<unsigned long long> mw;  // merged weights, node id nl + k
  mw.reserve(nl - 1);
  std::vector<int64_t> parent(2 * nl - 1, -1);
  int64_t li = 0, mi = 0;
  auto pop = [&]() -> std::pair<unsigned long long, int64_t> {
    const bool take_leaf = li < nl && (mi >= (int64_t)mw.size() || w[leaf[li]] <= mw[mi]);
    if (take_leaf) {
      const int64_t id = leaf[li++];
      return {w[id], id};
    }
    const int64_t id = nl + mi;
    return {mw[mi++], id};
  };
  for (int64_t k = 0; k < nl - 1; ++k) {
    const auto a = pop();
    const auto b = pop();
    parent[a.second] = nl + k;
    parent[b.second] = nl + k;
    mw.push_back(a.first + b.first);
  }
  const int64_t nid = 2 * nl - 1;
  std::vector<int> depth(nid, 0);
  for (int64_t node = nid - 2; node >= 0; --node) depth[node] = depth[parent[node]] + 1;  // parents come later
  for (int64_t i = 0; i < nl; ++i) len[present[i]] = (uint8_t)std::min(depth[i], 255);
  return len;
}

std::vector<uint8_t> huff_lengths(std::vector<unsigned long long> c) {
  for (;;) {
    std::vector<uint8_t> len = huff_tree_lengths(c);
    int mx = 0;
    for (uint8_t l : len) mx = std::max<int>(mx, l);
    if (mx <= kHuffMaxLen) return len;
    for (auto& v : c)
      if (v) v = (v + 1) / 2;
  }
}

// Canonical tables: cnt[l] codes of length l, first[l] the first of them, idx[l] the position
// of the first in `sorted` (symbols ordered by length, then value), code[s] every symbol's code.
struct HuffTables {
  uint32_t first[kHuffMaxLen + 1], cnt[kHuffMaxLen + 1], idx[kHuffMaxLen + 1];
  std::vector<int32_t> sorted;
  std::vector<uint32_t> code;
};

HuffTables huff_tables(const std::vector<uint8_t>& len) {
  HuffTables t;
  memset(t.first, 0, sizeof(t.first));
  memset(t.cnt, 0, sizeof(t.cnt));
  memset(t.idx, 0, sizeof(t.idx));
  for (uint8_t l : len)
    if (l) t.cnt[l]++;
  uint64_t code = 0;
  uint32_t pos = 0;
  for (int l = 1; l <= kHuffMaxLen; ++l) {
    code = (code + (l > 1 ? t.cnt[l - 1] : 0)) << (l > 1 ? 1 : 0);
    t.first[l] = (uint32_t)code;
    t.idx[l] = pos;
    pos += t.cnt[l];
  }
  t.sorted.assign(pos, 0);
  t.code.assign(len.size(), 0);
  uint32_t fill[kHuffMaxLen + 1];
  for (int l = 0; l <= kHuffMaxLen; ++l) fill[l] = 0;
  for (size_t s = 0; s < len.size(); ++s) {
    const int l = len[s];
    if (!l) continue;
    t.sorted[t.idx[l] + fill[l]] = (int32_t)s;
    t.code[s] = t.first[l] + fill[l];
    fill[l]++;
  }
  return t;
}

// Stream layout in the caller's output buffer: the header, the code lengths (nalpha bytes,
// padded to 16), the chunk offsets (uint64), then the 32-bit words.
struct HuffHeader {
  uint32_t magic, width;
  int64_t nsym, lo, nalpha, nbits, nchunks, pad[2];
};
constexpr uint32_t kHuffMagic = 0x46554846u;  // "FHUF"

struct HuffLayout {
  size_t off_len, off_chunks, off_words, bytes;
};
HuffLayout huff_layout(int64_t n, int64_t nalpha, int64_t nbits) {
  HuffLayout L;
  L.off_len = sizeof(HuffHeader);
  L.off_chunks = align_up(L.off_len + (size_t)nalpha, 16);
  const int64_t nch = (n + kHuffChunk - 1) / kHuffChunk;
  L.off_words = align_up(L.off_chunks + 8 * (size_t)nch, 16);
  L.bytes = L.off_words + 4 * (size_t)((nbits + 31) / 32);
  return L;
}

// Workspace: minmax partials, the frequency table, lengths, codes, block offsets, totals and
// the decoder's tables.
struct HuffWs {
  size_t off_mm, off_counts, off_code, off_boff, off_tot, off_tab, off_sorted, bytes;
};
// Whether a symbol stream starts on the 16-byte boundary that the kernels' vector accesses take.
int huff_vec(const void* p) { return ((uintptr_t)p & 15) == 0 ? 1 : 0; }

HuffWs huff_ws(int64_t n, int64_t nalpha) {
  HuffWs W;
  size_t off = 0;
  W.off_mm = off;
  off = align_up(off + 16 * 1024, 256);
  W.off_counts = off;
  off = align_up(off + 8 * (size_t)nalpha, 256);
  W.off_code = off;
  off = align_up(off + 4 * (size_t)nalpha, 256);
  const int64_t nblk = (n + kHuffBlockSyms - 1) / kHuffBlockSyms;
  W.off_boff = off;
  off = align_up(off + 8 * (size_t)std::max<int64_t>(1, nblk), 256);
  W.off_tot = off;
  off = align_up(off + 64, 256);
  // the decoder's upload: a zero status word, the sorted symbols
  W.off_tab = off;
  off += 16;
  W.off_sorted = off;
  off = align_up(off + 4 * (size_t)nalpha, 256);
  W.bytes = off;
  return W;
}

// Decode with the lengths compared rounded up to a multiple of 4.
template <int W>
hipError_t launch_huff_decode_w(int nl, const HuffDec& d, hipStream_t s) {
  const dim3 grid((unsigned)((d.nchunks + kHuffDecBlock - 1) / kHuffDecBlock)), block(kHuffDecBlock);
  const size_t dyn = 4 * (size_t)d.stage + 2 * (size_t)d.nlds;
  switch ((nl + 3) / 4) {
    case 1: hipLaunchKernelGGL((huff_decode_kernel<W, 4>), grid, block, dyn, s, d); break;
    case 2: hipLaunchKernelGGL((huff_decode_kernel<W, 8>), grid, block, dyn, s, d); break;
    case 3: hipLaunchKernelGGL((huff_decode_kernel<W, 12>), grid, block, dyn, s, d); break;
    case 4: hipLaunchKernelGGL((huff_decode_kernel<W, 16>), grid, block, dyn, s, d); break;
    case 5: hipLaunchKernelGGL((huff_decode_kernel<W, 20>), grid, block, dyn, s, d); break;
    case 6: hipLaunchKernelGGL((huff_decode_kernel<W, 24>), grid, block, dyn, s, d); break;
    default: hipLaunchKernelGGL((huff_decode_kernel<W, 33>), grid, block, dyn, s, d); break;
  }
  return hipGetLastError();
}
hipError_t launch_huff_decode(int width, int nl, const HuffDec& d, hipStream_t s) {
  return width == 1 ? launch_huff_decode_w<1>(nl, d, s) : launch_huff_decode_w<4>(nl, d, s);
}

// Scratch of ffcz_correct_noalloc (the array is declared at file scope, above): host
// code never passes the array's name to a kernel (on the host it names a host-side
// stand-in); it takes the device address hipGetSymbolAddress returns, once per device,
// with that device current.
constexpr int kMaxDevices = 64;
std::mutex g_scratch_m;
char* g_scratch_ptr[kMaxDevices] = {};

int32_t scratch_on_current_device(char** out) {
  int dev = -1;
  HIPCHK(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return fail(FFCZ_E_HIP, "device index beyond the scratch table");
  std::lock_guard<std::mutex> g(g_scratch_m);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    HIPCHK(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
    if (!ptr || ((uintptr_t)ptr & 255)) return fail(FFCZ_E_HIP, "scratch symbol address missing or misaligned");
    g_scratch_ptr[dev] = (char*)ptr;
  }
  *out = g_scratch_ptr[dev];
  return FFCZ_OK;
}

}  // namespace

extern "C" {

int32_t ffcz_version(void) { return 100; }

const char* ffcz_last_error(void) { return g_err.c_str(); }

int32_t ffcz_set_tuning(int32_t mode, const char* cache_path) {
  if (mode < 0 || mode > 4) return fail(FFCZ_E_INVALID, "tuning mode must be 0 to 4");
  std::lock_guard<std::mutex> g(g_tuner.m);
  g_tuner.init_locked();
  g_tuner.mode = mode;
  if (cache_path) {
    g_tuner.path = cache_path;
    g_tuner.loaded = false;
    g_tuner.load_locked();
  }
  return FFCZ_OK;
}

void ffcz_clear_tuning(void) {
  std::lock_guard<std::mutex> g(g_tuner.m);
  g_tuner.tab.clear();
  g_tuner.loaded = true;
}

int32_t ffcz_copy(void* dst, const void* src, size_t bytes, void* stream) {
  if (bytes == 0) return FFCZ_OK;
  if (!dst || !src) return fail(FFCZ_E_INVALID, "null pointer");
  if (((uintptr_t)dst & 15) || ((uintptr_t)src & 15)) return fail(FFCZ_E_INVALID, "pointers must be 16-byte aligned");
  hipStream_t s = (hipStream_t)stream;
  const int64_t n16 = (int64_t)(bytes / 16);
  if (n16 > 0) {
    for (int64_t v0 = 0; v0 < n16; v0 += (int64_t)1 << 36) {  // grid x holds 2^31 - 1 blocks
      const int64_t nv = std::min<int64_t>((int64_t)1 << 36, n16 - v0);
      hipLaunchKernelGGL(copy_kernel, dim3((unsigned)((nv + 255) / 256)), dim3(256), 0, s, (uint4*)dst + v0,
                         (const uint4*)src + v0, nv);
      HIPCHK(hipGetLastError());
    }
  }
  const int tail = (int)(bytes - (size_t)n16 * 16);
  if (tail > 0) {
    hipLaunchKernelGGL(copy_tail_kernel, dim3(1), dim3(16), 0, s, (unsigned char*)dst + n16 * 16,
                       (const unsigned char*)src + n16 * 16, tail);
    HIPCHK(hipGetLastError());
  }
  return FFCZ_OK;
}

int32_t ffcz_copy_columns(void* dst, const void* src, int64_t n_axis, int64_t axis_stride, int64_t n_fixed,
                          int64_t fixed_stride, int64_t row_bytes, void* stream) {
  if (n_axis < 0 || n_fixed < 0 || row_bytes < 0 || axis_stride < 0 || fixed_stride < 0)
    return fail(FFCZ_E_INVALID, "negative count, stride or row size");
  if (n_axis == 0 || n_fixed == 0 || row_bytes == 0) return FFCZ_OK;
  if (!dst || !src) return fail(FFCZ_E_INVALID, "null pointer");
  if ((((uintptr_t)dst | (uintptr_t)src) & 15) || ((axis_stride | fixed_stride | row_bytes) & 15))
    return fail(FFCZ_E_INVALID, "pointers, strides and the row size must be multiples of 16 bytes");
  const int64_t tiles = (row_bytes + 127) / 128;
  if (tiles > INT32_MAX || n_fixed > INT32_MAX / tiles) return fail(FFCZ_E_INVALID, "too many tiles for one launch");
  hipLaunchKernelGGL(copy_columns_kernel, dim3((unsigned)(n_fixed * tiles)), dim3(256), 0, (hipStream_t)stream,
                     (char*)dst, (const char*)src, n_axis, axis_stride, fixed_stride, row_bytes, (int32_t)tiles);
  HIPCHK(hipGetLastError());
  return FFCZ_OK;
}

void ffcz_profile_enable(int32_t on) {
  g_prof.on = on != 0;
  for (int k = 0; k < PK_COUNT; ++k) {
    g_prof.ms[k] = 0.0;
    g_prof.cnt[k] = 0;
  }
}

void ffcz_profile_select(uint32_t kinds) { g_prof.kinds = kinds; }

int32_t ffcz_profile_read(ffcz_profile* out) {
  if (!out) return fail(FFCZ_E_INVALID, "null pointer");
  for (auto& ev : g_prof.pending) {
    if (ev.keep == 1) {
      float ms = 0.f;
      if (hipEventSynchronize(ev.b) == hipSuccess && hipEventElapsedTime(&ms, ev.a, ev.b) == hipSuccess) {
        g_prof.ms[ev.kind] += ms;
        g_prof.cnt[ev.kind] += 1;
      }
    } else {
      (void)hipEventSynchronize(ev.b);
    }
    g_prof.pool.push_back(ev.a);
    g_prof.pool.push_back(ev.b);
  }
  g_prof.pending.clear();
  memset(out, 0, sizeof(*out));
  for (int k = 0; k < PK_COUNT && k < FFCZ_PROFILE_KINDS; ++k) {
    out->ms[k] = g_prof.ms[k];
    out->count[k] = g_prof.cnt[k];
    g_prof.ms[k] = 0.0;
    g_prof.cnt[k] = 0;
  }
  return FFCZ_OK;
}

void ffcz_default_options(ffcz_options* o) {
  if (!o) return;
  memset(o, 0, sizeof(*o));
  o->verify_fp64 = 1;
  o->graph_chunk = 4;
  o->use_graph = 1;
  o->resident_1d = 1;
  o->tiled_1d_lg = 0;
}

size_t ffcz_workspace_bytes(int32_t dtype, int32_t ndim, const int64_t* shape, int32_t max_iter) {
  if (route_1d(ndim, shape)) {
    const ffcz_instance in = one_instance(ndim, shape, nullptr, nullptr, nullptr, 0.0, 0.0);
    return ffcz_batched_workspace_bytes(dtype, 1, &in, max_iter < 0 ? 0 : max_iter);
  }
  Plan p;
  std::string keep = g_err;
  if (make_plan(dtype, ndim, shape, max_iter < 0 ? 0 : max_iter, 1, p) != FFCZ_OK) return 0;
  g_err = keep;
  return p.bytes;
}

size_t ffcz_mask_bytes(int32_t ndim, const int64_t* shape, int32_t rounds) {
  if (route_1d(ndim, shape)) return 0;  // the 1D signal path records no masks
  Plan p;
  std::string keep = g_err;
  if (rounds < 0 || make_plan(FFCZ_F32, ndim, shape, rounds, 1, p) != FFCZ_OK) return 0;
  g_err = keep;
  return (size_t)(rounds + 1) * p.s_plane_bytes + (size_t)rounds * 2 * p.f_plane_bytes;
}

int32_t ffcz_suggest_margin(int32_t dtype, int32_t ndim, const int64_t* shape, const void* x, double delta_f,
                            void* ws, size_t ws_bytes, void* stream, double* mu_out) {
  int64_t N = 1;
  if (route_1d(ndim, shape)) {
    int64_t sq[3];
    const int nd = squeeze(ndim, shape, sq);
    if (nd == 1) N = sq[0];
    if (N > (int64_t)1 << 19) return fail(FFCZ_E_SHAPE, "1D lengths must be at most 2^19");
    if (dtype != FFCZ_F32 && dtype != FFCZ_F64) return fail(FFCZ_E_INVALID, "dtype must be FFCZ_F32 or FFCZ_F64");
  } else {
    Plan p;
    int32_t r = make_plan(dtype, ndim, shape, 0, 1, p);
    if (r != FFCZ_OK) return r;
    N = p.N;
  }
  if (!x || !mu_out) return fail(FFCZ_E_INVALID, "null pointer");
  if (!std::isfinite(delta_f) || delta_f < 0) return fail(FFCZ_E_INVALID, "delta_f must be finite and >= 0");
  if (dtype == FFCZ_F64) {
    *mu_out = std::ldexp(1.0, -16);
    return FFCZ_OK;
  }
  // the reduction's slots sit at the start of the workspace
  if (!ws || ws_bytes < sizeof(double) * (kUlpSlots + 1) || ((uintptr_t)ws & 255))
    return fail(FFCZ_E_WORKSPACE, "workspace too small or misaligned");
  hipStream_t s = (hipStream_t)stream;
  double* slots = (double*)ws;
  const int nsl = ulp_slots(N);
  const MarginJob job{(const float*)x, N, delta_f, 0};
  hipLaunchKernelGGL(ulp_part_kernel, dim3((unsigned)nsl), dim3(256), 0, s, job, (const MarginJob*)nullptr, slots);
  HIPCHK(hipGetLastError());
  hipLaunchKernelGGL(margin_kernel, dim3(1), dim3(256), 0, s, (const double*)slots, job,
                     (const MarginJob*)nullptr, (int)FFCZ_F32, slots + kUlpSlots, (DevState*)nullptr);
  HIPCHK(hipGetLastError());
  HIPCHK(g_host_misc.reserve(sizeof(double)));
  HIPCHK(hipMemcpyAsync(g_host_misc.p, slots + kUlpSlots, sizeof(double), hipMemcpyDeviceToHost, s));
  HIPCHK(hipStreamSynchronize(s));
  *mu_out = *(const double*)g_host_misc.p;
  return FFCZ_OK;
}

int32_t ffcz_correct(int32_t dtype, int32_t ndim, const int64_t* shape, const void* x, const void* xb, void* y,
                     double eps_s, double delta_f, int32_t max_iter, const ffcz_options* opts, void* ws,
                     size_t ws_bytes, void* stream, ffcz_stats* stats) {
  if (route_1d(ndim, shape)) {
    // one signal of any length on the 1D path, as a batch of one
    if (opts && (opts->masks_out || opts->viol_per_round))
      return fail(FFCZ_E_INVALID, "masks and per-check counts are recorded for power-of-two fields only");
    if (!x || !xb || !y) return fail(FFCZ_E_INVALID, "null data pointer");
    const ffcz_instance in = one_instance(ndim, shape, x, xb, y, eps_s, delta_f);
    ffcz_stats st;
    memset(&st, 0, sizeof(st));
    const int32_t r = ffcz_correct_batched(dtype, 1, &in, max_iter, opts, ws, ws_bytes, stream, &st);
    if (r == FFCZ_E_NONFINITE) g_err = "x or x_hat holds NaN or Inf";
    if (stats && st.status == r) *stats = st;
    return r;
  }
  SingleCall sc;
  int32_t r = single_setup(dtype, ndim, shape, x, xb, y, eps_s, delta_f, max_iter, opts, sc);
  if (r != FFCZ_OK) return r;
  if (!ws || ws_bytes < sc.p.bytes) return fail(FFCZ_E_WORKSPACE, "workspace smaller than ffcz_workspace_bytes()");
  if ((uintptr_t)ws & 255) return fail(FFCZ_E_WORKSPACE, "workspace must be 256-byte and data 16-byte aligned");
  return single_run(sc, (char*)ws, (hipStream_t)stream, stats, nullptr);
}

int32_t ffcz_correct_noalloc(int32_t dtype, int32_t ndim, const int64_t* shape, const void* x, const void* xb,
                             void* y, double eps_s, double delta_f, int32_t max_iter, const ffcz_options* opts,
                             void* stream, ffcz_stats* stats) {
  if (route_1d(ndim, shape))
    return fail(FFCZ_E_SHAPE, "ffcz_correct_noalloc takes power-of-two fields only (the 1D signal path stages "
                              "its descriptors in pinned host memory)");
  SingleCall sc;
  int32_t r = single_setup(dtype, ndim, shape, x, xb, y, eps_s, delta_f, max_iter, opts, sc);
  if (r != FFCZ_OK) return r;
  if (sc.p.bytes > kScratchBytes)
    return fail(FFCZ_E_WORKSPACE, "ffcz_correct_noalloc: this shape and round cap need " +
                                      std::to_string(sc.p.bytes) + " bytes of scratch, above the fixed " +
                                      std::to_string(kScratchBytes) + " (FFCZ_NOALLOC_SCRATCH_BYTES)");
  char* ws = nullptr;
  r = scratch_on_current_device(&ws);
  if (r != FFCZ_OK) return r;
  DevState host_state;  // the loop state is read back into this (no pinned staging)
  return single_run(sc, ws, (hipStream_t)stream, stats, &host_state);
}

size_t ffcz_bounds_workspace_bytes(int32_t dtype, int32_t ndim, const int64_t* shape, int32_t max_iter) {
  if (route_1d(ndim, shape)) return 0;
  Plan p;
  std::string keep = g_err;
  if (make_plan(dtype, ndim, shape, max_iter < 0 ? 0 : max_iter, 1, p) != FFCZ_OK) return 0;
  g_err = keep;
  return bounds_layout(p).bytes;
}

int32_t ffcz_correct_bounds(int32_t dtype, int32_t ndim, const int64_t* shape, const void* x, const void* xb,
                            void* y, double eps_s, double delta_f, const ffcz_bounds* bnd, int32_t max_iter,
                            const ffcz_options* opts, void* ws, size_t ws_bytes, void* stream, ffcz_stats* stats) {
  if (route_1d(ndim, shape))
    return fail(FFCZ_E_SHAPE, "pointwise bounds take fields that run on the multidimensional passes");
  SingleCall sc;
  int32_t r = single_setup(dtype, ndim, shape, x, xb, y, eps_s, delta_f, max_iter, opts, sc);
  if (r != FFCZ_OK) return r;
  if (sc.o.masks_out) return fail(FFCZ_E_INVALID, "masks are not recorded with pointwise bounds");
  ffcz_bounds b;
  memset(&b, 0, sizeof(b));
  if (bnd) b = *bnd;
  if (((uintptr_t)b.eps_s & 15) || ((uintptr_t)b.delta_re & 15) || ((uintptr_t)b.delta_im & 15))
    return fail(FFCZ_E_WORKSPACE, "bound arrays must be 16-byte aligned");
  const BoundsLayout L = bounds_layout(sc.p);
  if (!ws || ws_bytes < L.bytes) return fail(FFCZ_E_WORKSPACE, "workspace smaller than ffcz_bounds_workspace_bytes()");
  if ((uintptr_t)ws & 255) return fail(FFCZ_E_WORKSPACE, "workspace must be 256-byte aligned");
  char* w = (char*)ws;
  BoundsCfg bc;
  bc.pE = b.eps_s;
  bc.disk = b.disk ? 1 : 0;
  bc.dre = b.delta_re;
  bc.dim = bc.disk ? b.delta_re : b.delta_im;  // the disk bounds the modulus by delta_re
  bc.sre = delta_f;
  bc.sim = delta_f;
  bc.pD = w + L.off_D;
  bc.minpart = (unsigned long long*)(w + L.off_min);
  bc.bad = (unsigned long long*)(w + L.off_bad);
  const double* mus = sc.mu > 0.0 && sc.o.margin_rel > 0.0 ? &sc.mu : nullptr;
  hipStream_t s = (hipStream_t)stream;
  int32_t status = FFCZ_OK;
  r = dtype == FFCZ_F32 ? correct_group<float>(sc.p, &sc.in, mus, max_iter, sc.o, w, s, stats, &status, nullptr,
                                               nullptr, &bc)
                        : correct_group<double>(sc.p, &sc.in, mus, max_iter, sc.o, w, s, stats, &status, nullptr,
                                                nullptr, &bc);
  if (r != FFCZ_OK) return r;
  if (stats) stats->status = status;
  if (status == FFCZ_E_NONFINITE) return fail(FFCZ_E_NONFINITE, "x or x_hat holds NaN or Inf");
  if (status == FFCZ_VERIFY_FAILED) g_err = "FP64 re-verification against the pointwise bounds failed";
  return status;
}

int32_t ffcz_power_spectrum_bounds(int32_t dtype, int32_t ndim, const int64_t* shape, const void* x, double rho,
                                   int32_t disk, void* delta_out, void* ws, size_t ws_bytes, void* stream) {
  if (route_1d(ndim, shape))
    return fail(FFCZ_E_SHAPE, "power-spectrum bounds take fields that run on the multidimensional passes");
  Plan p;
  int32_t r = make_plan(dtype, ndim, shape, 0, 1, p);
  if (r != FFCZ_OK) return r;
  if (!x || !delta_out) return fail(FFCZ_E_INVALID, "null pointer");
  if (!std::isfinite(rho) || rho < 0) return fail(FFCZ_E_INVALID, "rho must be finite and >= 0");
  if (((uintptr_t)x & 15) || ((uintptr_t)delta_out & 15)) return fail(FFCZ_E_WORKSPACE, "data must be 16-byte aligned");
  const BoundsLayout L = bounds_layout(p);
  if (L.nb > kMaxShells) return fail(FFCZ_E_SHAPE, "too many shells");
  if (!ws || ws_bytes < L.bytes) return fail(FFCZ_E_WORKSPACE, "workspace smaller than ffcz_bounds_workspace_bytes()");
  if ((uintptr_t)ws & 255) return fail(FFCZ_E_WORKSPACE, "workspace must be 256-byte aligned");
  hipStream_t s = (hipStream_t)stream;
  return dtype == FFCZ_F32 ? power_bounds_impl<float>(p, L, (char*)ws, x, rho, disk ? 1 : 0, delta_out, s)
                           : power_bounds_impl<double>(p, L, (char*)ws, x, rho, disk ? 1 : 0, delta_out, s);
}

size_t ffcz_huffman_workspace_bytes(int64_t nsym, int64_t nalpha) {
  if (nsym < 0 || nalpha < 0 || nalpha > kHuffMaxAlpha) return 0;
  return huff_ws(nsym, nalpha).bytes;
}

int32_t ffcz_huffman_plan(const void* sym, int64_t nsym, int32_t width, void* ws, size_t ws_bytes, void* stream,
                          ffcz_huffman_sizes* plan) {
  if (!plan || (nsym > 0 && !sym)) return fail(FFCZ_E_INVALID, "null pointer");
  if (width != 1 && width != 4) return fail(FFCZ_E_INVALID, "width must be 1 or 4");
  if (nsym < 0) return fail(FFCZ_E_INVALID, "nsym must be >= 0");
  memset(plan, 0, sizeof(*plan));
  plan->nsym = nsym;
  if (nsym > 0) {
    if (!ws || ws_bytes < huff_ws(nsym, 0).bytes || ((uintptr_t)ws & 255))
      return fail(FFCZ_E_WORKSPACE, "workspace smaller than ffcz_huffman_workspace_bytes(nsym, 0) or misaligned");
    hipStream_t s = (hipStream_t)stream;
    const int g = (int)std::min<int64_t>(1024, (nsym + kHuffBlockSyms - 1) / kHuffBlockSyms);
    long long* mm = (long long*)ws;
    const auto kern = width == 1 ? huff_minmax_kernel<1> : huff_minmax_kernel<4>;
    hipLaunchKernelGGL(kern, dim3((unsigned)g), dim3(kHuffBlock), 0, s, sym, nsym, huff_vec(sym), mm);
    HIPCHK(hipGetLastError());
    HIPCHK(g_host_misc.reserve(2 * sizeof(long long) * (size_t)g));
    const long long* h = (const long long*)g_host_misc.p;
    HIPCHK(hipMemcpyAsync(g_host_misc.p, mm, 2 * sizeof(long long) * (size_t)g, hipMemcpyDeviceToHost, s));
    HIPCHK(hipStreamSynchronize(s));
    long long lo = h[0], hi = h[1];
    for (int b = 1; b < g; ++b) {
      lo = std::min(lo, h[2 * b]);
      hi = std::max(hi, h[2 * b + 1]);
    }
    plan->lo = lo;
    plan->nalpha = hi - lo + 1;
    if (plan->nalpha > kHuffMaxAlpha) return fail(FFCZ_E_INVALID, "alphabet wider than 2^24 symbols");
  }
  plan->ws_bytes = huff_ws(nsym, plan->nalpha).bytes;
  plan->out_bytes = huff_layout(nsym, plan->nalpha, 32 * nsym).bytes;
  return FFCZ_OK;
}

int32_t ffcz_huffman_encode(const void* sym, int64_t nsym, int32_t width, const ffcz_huffman_sizes* plan, void* out,
                            size_t out_bytes, void* ws, size_t ws_bytes, void* stream, size_t* used_bytes) {
  if (!plan || !out || (nsym > 0 && !sym)) return fail(FFCZ_E_INVALID, "null pointer");
  if (width != 1 && width != 4) return fail(FFCZ_E_INVALID, "width must be 1 or 4");
  if (plan->nsym != nsym || plan->nalpha < 0 || plan->nalpha > kHuffMaxAlpha)
    return fail(FFCZ_E_INVALID, "plan does not match the stream");
  if ((uintptr_t)out & 15) return fail(FFCZ_E_WORKSPACE, "output must be 16-byte aligned");
  const int64_t nalpha = plan->nalpha, lo = plan->lo;
  const HuffWs W = huff_ws(nsym, nalpha);
  if (!ws || ws_bytes < W.bytes || ((uintptr_t)ws & 255))
    return fail(FFCZ_E_WORKSPACE, "workspace smaller than the plan's ws_bytes or misaligned");
  hipStream_t s = (hipStream_t)stream;
  char* w = (char*)ws;
  char* o = (char*)out;
  HuffHeader hd;
  memset(&hd, 0, sizeof(hd));
  hd.magic = kHuffMagic;
  hd.width = (uint32_t)width;
  hd.nsym = nsym;
  hd.lo = lo;
  hd.nalpha = nalpha;
  hd.nchunks = (nsym + kHuffChunk - 1) / kHuffChunk;
  const int vec = huff_vec(sym);
  const bool w1 = width == 1;
  HuffTables t;
  std::vector<uint8_t> len;
  if (nsym > 0) {
    // the global frequency table, then the code on the host
    unsigned long long* counts = (unsigned long long*)(w + W.off_counts);
    hipLaunchKernelGGL(zero_u64_kernel, dim3((unsigned)((nalpha + 255) / 256)), dim3(256), 0, s, counts, nalpha);
    HIPCHK(hipGetLastError());
    // with a table in LDS, at most one block per CU, of at least two groups (each adds its table at
    // the end); straight into memory, a block a group (1 M codes over 57 K symbols: 65 -> 59 us)
    const int64_t group = (int64_t)kHuffHistBlock * kHuffPerLane;
    const bool local = nalpha <= kHuffLdsBins;
    const int g = (int)std::max<int64_t>(1, local ? std::min<int64_t>(256, nsym / (2 * group))
                                                  : std::min<int64_t>(1024, (nsym + group - 1) / group));
    const size_t bins = local ? 4 * (size_t)nalpha : 0;
    hipLaunchKernelGGL(w1 ? huff_hist_kernel<1> : huff_hist_kernel<4>, dim3((unsigned)g), dim3(kHuffHistBlock), bins,
                       s, sym, nsym, (int64_t)lo, nalpha, vec, counts);
    HIPCHK(hipGetLastError());
    // through pinned staging: the table out, then header, lengths and codes back (copied in by the
    // synchronisation at the end, before the buffer is reused)
    HIPCHK(g_host_misc.reserve(std::max(8 * (size_t)nalpha, sizeof(hd) + 5 * (size_t)nalpha + 16)));
    unsigned long long* hcp = (unsigned long long*)g_host_misc.p;
    HIPCHK(hipMemcpyAsync(hcp, counts, 8 * (size_t)nalpha, hipMemcpyDeviceToHost, s));
    HIPCHK(hipStreamSynchronize(s));
    const std::vector<unsigned long long> freq(hcp, hcp + nalpha);
    len = huff_lengths(freq);
    t = huff_tables(len);
    unsigned long long nbits = 0;
    for (int64_t i = 0; i < nalpha; ++i) nbits += freq[i] * len[i];
    hd.nbits = (int64_t)nbits;
  }
  const HuffLayout L = huff_layout(nsym, nalpha, hd.nbits);
  if (out_bytes < L.bytes)
    return fail(FFCZ_E_WORKSPACE, "output smaller than the stream (" + std::to_string(L.bytes) + " bytes)");
  HIPCHK(g_host_misc.reserve(sizeof(hd) + 5 * (size_t)nalpha + 16));
  char* const hb = (char*)g_host_misc.p;
  memcpy(hb, &hd, sizeof(hd));
  if (nsym > 0) memcpy(hb + L.off_len, len.data(), (size_t)nalpha);
  HIPCHK(hipMemcpyAsync(o, hb, L.off_len + (nsym > 0 ? (size_t)nalpha : 0), hipMemcpyHostToDevice, s));
  if (nsym > 0) {
    uint32_t* dcode = (uint32_t*)(w + W.off_code);
    uint32_t* hcode = (uint32_t*)(hb + align_up(L.off_len + (size_t)nalpha, 16));
    memcpy(hcode, t.code.data(), 4 * (size_t)nalpha);
    HIPCHK(hipMemcpyAsync(dcode, hcode, 4 * (size_t)nalpha, hipMemcpyHostToDevice, s));
    const uint8_t* dlen = (const uint8_t*)(o + L.off_len);
    // bits per block and block offsets
    const int64_t nblk = (nsym + kHuffBlockSyms - 1) / kHuffBlockSyms;
    unsigned long long* boff = (unsigned long long*)(w + W.off_boff);
    unsigned long long* tot = (unsigned long long*)(w + W.off_tot);
    hipLaunchKernelGGL(w1 ? huff_bits_kernel<1> : huff_bits_kernel<4>, dim3((unsigned)nblk), dim3(kHuffBlock), 0, s,
                       sym, nsym, (int64_t)lo, nalpha, vec, dlen, boff);
    HIPCHK(hipGetLastError());
    hipLaunchKernelGGL(edit_scan_kernel, dim3(1), dim3(1024), 0, s, ScanJob{boff, nblk, tot}, ScanJob{},
                       (unsigned*)nullptr);
    HIPCHK(hipGetLastError());
    const int64_t nwords = (hd.nbits + 31) / 32;
    hipLaunchKernelGGL(zero_u32_kernel, dim3((unsigned)((nwords + 255) / 256)), dim3(256), 0, s,
                       (uint32_t*)(o + L.off_words), nwords);
    HIPCHK(hipGetLastError());
    hipLaunchKernelGGL(w1 ? huff_encode_kernel<1> : huff_encode_kernel<4>, dim3((unsigned)nblk), dim3(kHuffBlock), 0,
                       s, sym, nsym, (int64_t)lo, nalpha, vec, dlen, (const uint32_t*)dcode,
                       (const unsigned long long*)boff, (unsigned int*)(o + L.off_words),
                       (unsigned long long*)(o + L.off_chunks));
    HIPCHK(hipGetLastError());
  }
  HIPCHK(hipStreamSynchronize(s));
  if (used_bytes) *used_bytes = L.bytes;
  return FFCZ_OK;
}

int32_t ffcz_huffman_decode(const void* in, size_t in_bytes, int32_t width, void* sym_out, int64_t capacity, void* ws,
                            size_t ws_bytes, void* stream, int64_t* nsym_out) {
  if (!in || in_bytes < sizeof(HuffHeader)) return fail(FFCZ_E_INVALID, "input too short");
  if ((uintptr_t)in & 15) return fail(FFCZ_E_WORKSPACE, "input must be 16-byte aligned");
  hipStream_t s = (hipStream_t)stream;
  // the header and, where they are short, the lengths after it in one read (pinned staging)
  const size_t head = std::min<size_t>(in_bytes, 16384);
  HIPCHK(g_host_misc.reserve(16384));
  HIPCHK(hipMemcpyAsync(g_host_misc.p, in, head, hipMemcpyDeviceToHost, s));
  HIPCHK(hipStreamSynchronize(s));
  HuffHeader hd;
  memcpy(&hd, g_host_misc.p, sizeof(hd));
  if (hd.magic != kHuffMagic || (hd.width != 1 && hd.width != 4) || hd.nsym < 0 || hd.nalpha < 0 ||
      hd.nalpha > kHuffMaxAlpha || hd.nbits < 0)
    return fail(FFCZ_E_INVALID, "not a stream written by ffcz_huffman_encode");
  if ((int32_t)hd.width != width) return fail(FFCZ_E_INVALID, "symbol width differs from the stream's");
  if (hd.nchunks != (hd.nsym + kHuffChunk - 1) / kHuffChunk)
    return fail(FFCZ_E_INVALID, "chunk count does not match the symbol count");
  const HuffLayout L = huff_layout(hd.nsym, hd.nalpha, hd.nbits);
  if (in_bytes < L.bytes) return fail(FFCZ_E_INVALID, "input shorter than its stream");
  if (hd.nsym > capacity || (hd.nsym > 0 && !sym_out)) return fail(FFCZ_E_INVALID, "output holds fewer symbols than the stream");
  if (nsym_out) *nsym_out = hd.nsym;
  if (hd.nsym == 0) return FFCZ_OK;
  const HuffWs W = huff_ws(hd.nsym, hd.nalpha);
  if (!ws || ws_bytes < W.bytes || ((uintptr_t)ws & 255))
    return fail(FFCZ_E_WORKSPACE, "workspace smaller than ffcz_huffman_workspace_bytes(nsym, nalpha) or misaligned");
  const char* ib = (const char*)in;
  std::vector<uint8_t> len((size_t)hd.nalpha);
  if (L.off_len + (size_t)hd.nalpha <= head) {
    memcpy(len.data(), (const char*)g_host_misc.p + L.off_len, (size_t)hd.nalpha);
  } else {
    HIPCHK(g_host_misc.reserve((size_t)hd.nalpha));
    HIPCHK(hipMemcpyAsync(g_host_misc.p, ib + L.off_len, (size_t)hd.nalpha, hipMemcpyDeviceToHost, s));
    HIPCHK(hipStreamSynchronize(s));
    memcpy(len.data(), g_host_misc.p, (size_t)hd.nalpha);
  }
  for (uint8_t l : len)
    if (l > kHuffMaxLen) return fail(FFCZ_E_INVALID, "code length above 32 in the stream");
  const HuffTables t = huff_tables(len);
  // a prefix code: at most 2^l codes of length l after the shorter ones (Kraft), so every
  // window the decoder meets maps into the table or is reported
  uint64_t kraft = 0;  // sum of 2^(32 - l) over the codes, at most 2^32
  for (int l = 1; l <= kHuffMaxLen; ++l) kraft += (uint64_t)t.cnt[l] << (kHuffMaxLen - l);
  if (kraft > (1ull << kHuffMaxLen)) return fail(FFCZ_E_INVALID, "code lengths break the Kraft inequality");
  char* w = (char*)ws;
  // a zero status word and the sorted symbols (one upload)
  const size_t up = W.off_sorted + 4 * t.sorted.size() - W.off_tab;
  HIPCHK(g_host_misc.reserve(up));
  memset(g_host_misc.p, 0, W.off_sorted - W.off_tab);
  if (!t.sorted.empty())
    memcpy((char*)g_host_misc.p + (W.off_sorted - W.off_tab), t.sorted.data(), 4 * t.sorted.size());
  HIPCHK(hipMemcpyAsync(w + W.off_tab, g_host_misc.p, up, hipMemcpyHostToDevice, s));
  unsigned int* bad = (unsigned int*)(w + W.off_tab);
  HuffDec d;
  memset(&d, 0, sizeof(d));
  d.words = (const unsigned int*)(ib + L.off_words);
  d.nwords = (hd.nbits + 31) / 32;
  d.chunk_bits = (const unsigned long long*)(ib + L.off_chunks);
  d.nbits = (unsigned long long)hd.nbits;
  d.n = hd.nsym;
  d.lo = hd.lo;
  d.nchunks = hd.nchunks;
  d.sorted = (const int32_t*)(w + W.off_sorted);
  int lmin = 0, lmax = 0;
  for (int l = 1; l <= kHuffMaxLen; ++l)
    if (t.cnt[l]) {
      if (!lmin) lmin = l;
      lmax = l;
    }
  if (!lmin) return fail(FFCZ_E_INVALID, "the stream has symbols but no codes");
  d.lmin = lmin;
  d.nlen = lmax - lmin + 1;
  d.nsorted = (int32_t)t.sorted.size();
  for (int j = 0; j < 32; ++j) d.top[j] = 0xffffffffu;
  uint64_t lim = 0;
  for (int l = lmin; l <= lmax; ++l) {
    lim = ((uint64_t)t.first[l] + t.cnt[l]) << (32 - l);  // left-justified end of the codes up to length l
    d.top[l - lmin] = (uint32_t)(lim - 1);
    d.off[l - lmin] = t.idx[l] - t.first[l];
  }
  // lengths compared: those of the code, and one more that catches the patterns of an incomplete code
  const int nl = d.nlen + (lim < (1ull << 32) ? 1 : 0);
  // words staged per block: all that its chunks can hold, at most 48 KB, and no more than twice
  // what they hold on average (more blocks per CU; a wave with a longer stretch reads memory)
  const int64_t most = (int64_t)kHuffDecBlock * kHuffChunk * lmax / 32 + 4;
  const int64_t mean = (hd.nbits / std::max<int64_t>(1, hd.nchunks) + 1) * kHuffDecBlock / 32;
  d.stage = (int)std::min<int64_t>(12288, std::min(most, 2 * mean + 64));
  // the symbols in LDS where they fit in 64 KB
  d.nlds = t.sorted.size() <= 32768 && hd.nalpha <= 65536 ? (int)t.sorted.size() : 0;
  d.vec = huff_vec(sym_out);
  d.out = sym_out;
  d.bad = bad;
  HIPCHK(launch_huff_decode(width, nl, d, s));
  HIPCHK(hipMemcpyAsync(g_host_misc.p, bad, 4, hipMemcpyDeviceToHost, s));
  HIPCHK(hipStreamSynchronize(s));
  const unsigned int hb = *(const unsigned int*)g_host_misc.p;
  if (hb) return fail(FFCZ_E_INVALID, "the stream holds a bit pattern that is no code");
  return FFCZ_OK;
}

size_t ffcz_encode_workspace_bytes(int32_t dtype, int32_t ndim, const int64_t* shape, int32_t max_iter) {
  if (route_1d(ndim, shape)) return 0;
  Plan p;
  std::string keep = g_err;
  if (make_plan(dtype, ndim, shape, max_iter < 0 ? 0 : max_iter, 1, p) != FFCZ_OK) return 0;
  g_err = keep;
  return edit_layout(p).bytes;
}

void ffcz_default_encode_options(ffcz_encode_options* o) {
  if (!o) return;
  memset(o, 0, sizeof(*o));
  o->m = 16;
  o->safety = 4.0;
}

int32_t ffcz_encode(int32_t dtype, int32_t ndim, const int64_t* shape, const void* x, const void* xb, double eps_s,
                    double delta_f, int32_t max_iter, const ffcz_options* opts, const ffcz_encode_options* eopts,
                    void* spat_flags, int32_t* spat_codes, void* freq_flags, int32_t* freq_codes, void* ws,
                    size_t ws_bytes, void* stream, ffcz_encode_stats* est) {
  if (route_1d(ndim, shape))
    return fail(FFCZ_E_SHAPE, "the encoder takes fields that run on the multidimensional passes (power-of-two extents)");
  ffcz_encode_options eo;
  if (eopts) eo = *eopts;
  else ffcz_default_encode_options(&eo);
  const int m = eo.m > 0 ? eo.m : 16;
  const double safety = eo.safety > 0.0 ? eo.safety : 4.0;
  if (m > 30) return fail(FFCZ_E_INVALID, "code length m must be at most 30");
  if (!std::isfinite(safety)) return fail(FFCZ_E_INVALID, "safety must be finite");
  if (!(eo.mu_s >= 0.0 && eo.mu_s < 0.5) || !(eo.mu_f >= 0.0 && eo.mu_f < 0.25))
    return fail(FFCZ_E_INVALID, "mu_s must lie in [0, 1/2) and mu_f in [0, 1/4)");
  if ((eo.mu_s > 0.0) != (eo.mu_f > 0.0)) return fail(FFCZ_E_INVALID, "give both shrinks or neither");
  SingleCall sc;
  // without y_out the closing pass does not run and nothing is written to the output pointer
  void* y = eo.y_out ? eo.y_out : const_cast<void*>(xb);
  int32_t r = single_setup(dtype, ndim, shape, x, xb, y, eps_s, delta_f, max_iter, opts, sc);
  if (r != FFCZ_OK) return r;
  if (!spat_flags || !spat_codes || !freq_flags || !freq_codes) return fail(FFCZ_E_INVALID, "null flag or code buffer");
  if (((uintptr_t)spat_flags & 15) || ((uintptr_t)spat_codes & 15) || ((uintptr_t)freq_flags & 15) ||
      ((uintptr_t)freq_codes & 15) || ((uintptr_t)eo.spat_edits_out & 15) || ((uintptr_t)eo.freq_edits_out & 15))
    return fail(FFCZ_E_WORKSPACE, "flag, code and edit buffers must be 16-byte aligned");
  const EditLayout L = edit_layout(sc.p);
  if (!ws || ws_bytes < L.bytes) return fail(FFCZ_E_WORKSPACE, "workspace smaller than ffcz_encode_workspace_bytes()");
  if ((uintptr_t)ws & 255) return fail(FFCZ_E_WORKSPACE, "workspace must be 256-byte aligned");
  if (!eo.y_out) sc.o.verify_fp64 = 0;
  char* w = (char*)ws;
  EditCfg ed;
  ed.sacc = w + L.off_S;
  ed.facc = w + L.off_F;
  ed.derive = eo.mu_s == 0.0;
  ed.q = safety * std::ldexp(1.0, -m);
  ed.mu_s = eo.mu_s;
  ed.mu_f = eo.mu_f;
  ed.want_y = eo.y_out != nullptr;
  ed.amax = (unsigned long long*)(w + L.off_amax);
  double mu_s_used = 0.0;
  ed.mu_s_out = &mu_s_used;
  sc.mu = 0.5;  // placeholder: the encoder's own shrinks replace the margin (on the host or the device)
  hipStream_t s = (hipStream_t)stream;
  ffcz_stats lst;
  memset(&lst, 0, sizeof(lst));
  int32_t status = FFCZ_OK;
  const double* mus = &sc.mu;
  r = dtype == FFCZ_F32 ? correct_group<float>(sc.p, &sc.in, mus, max_iter, sc.o, w, s, &lst, &status, nullptr, &ed)
                        : correct_group<double>(sc.p, &sc.in, mus, max_iter, sc.o, w, s, &lst, &status, nullptr, &ed);
  if (r != FFCZ_OK) return r;
  lst.status = status;
  if (status == FFCZ_E_NONFINITE) return fail(FFCZ_E_NONFINITE, "x or x_hat holds NaN or Inf");
  const double step_s = std::ldexp(2.0 * eps_s, -m), step_f = std::ldexp(2.0 * delta_f, -m);
  int64_t nnz_s = 0, nnz_f = 0;
  r = dtype == FFCZ_F32 ? code_edits<float>(sc.p, L, w, spat_flags, spat_codes, freq_flags, freq_codes, step_s,
                                            step_f, eo.spat_edits_out, eo.freq_edits_out, s, &nnz_s, &nnz_f)
                        : code_edits<double>(sc.p, L, w, spat_flags, spat_codes, freq_flags, freq_codes, step_s,
                                             step_f, eo.spat_edits_out, eo.freq_edits_out, s, &nnz_s, &nnz_f);
  if (r != FFCZ_OK) return r;
  if (est) {
    memset(est, 0, sizeof(*est));
    est->loop = lst;
    est->nnz_s = nnz_s;
    est->nnz_f = nnz_f;
    est->step_s = step_s;
    est->step_f = step_f;
    // the shrinks in use: the state read back by the loop
    est->mu_f = lst.margin_used;
    est->mu_s = mu_s_used;
    est->m = m;
    est->status = status;
  }
  if (status == FFCZ_VERIFY_FAILED) g_err = "FP64 re-verification of y failed";
  return status;
}

int32_t ffcz_decode(int32_t dtype, int32_t ndim, const int64_t* shape, const void* xb, const void* spat_flags,
                    const int32_t* spat_codes, int64_t nnz_s, const void* freq_flags, const int32_t* freq_codes,
                    int64_t nnz_f, double step_s, double step_f, void* y, void* ws, size_t ws_bytes, void* stream) {
  if (route_1d(ndim, shape))
    return fail(FFCZ_E_SHAPE, "the decoder takes fields that run on the multidimensional passes (power-of-two extents)");
  Plan p;
  int32_t r = make_plan(dtype, ndim, shape, 0, 1, p);
  if (r != FFCZ_OK) return r;
  const EditLayout L = edit_layout(p);
  if (!xb || !y || !spat_flags || !freq_flags) return fail(FFCZ_E_INVALID, "null pointer");
  if ((nnz_s > 0 && !spat_codes) || (nnz_f > 0 && !freq_codes)) return fail(FFCZ_E_INVALID, "null code buffer");
  if (nnz_s < 0 || nnz_f < 0 || nnz_s > L.ncs || nnz_f > L.ncf) return fail(FFCZ_E_INVALID, "code counts out of range");
  if (xb == y) return fail(FFCZ_E_INVALID, "x_base and y must not alias");
  if (!std::isfinite(step_s) || !std::isfinite(step_f) || step_s < 0 || step_f < 0)
    return fail(FFCZ_E_INVALID, "steps must be finite and >= 0");
  if (((uintptr_t)xb & 15) || ((uintptr_t)y & 15) || ((uintptr_t)spat_flags & 15) || ((uintptr_t)freq_flags & 15) ||
      ((uintptr_t)spat_codes & 15) || ((uintptr_t)freq_codes & 15))
    return fail(FFCZ_E_WORKSPACE, "data, flag and code buffers must be 16-byte aligned");
  if (!ws || ws_bytes < L.bytes) return fail(FFCZ_E_WORKSPACE, "workspace smaller than ffcz_encode_workspace_bytes()");
  if ((uintptr_t)ws & 255) return fail(FFCZ_E_WORKSPACE, "workspace must be 256-byte aligned");
  hipStream_t s = (hipStream_t)stream;
  return dtype == FFCZ_F32 ? decode_impl<float>(p, L, (char*)ws, xb, spat_flags, spat_codes, nnz_s, freq_flags,
                                                freq_codes, nnz_f, step_s, step_f, y, s)
                           : decode_impl<double>(p, L, (char*)ws, xb, spat_flags, spat_codes, nnz_s, freq_flags,
                                                 freq_codes, nnz_f, step_s, step_f, y, s);
}

size_t ffcz_batched_workspace_bytes(int32_t dtype, int32_t count, const ffcz_instance* inst, int32_t max_iter) {
  BatchPlan bp;
  std::string keep = g_err;
  if (max_iter < 0 || batch_plan(dtype, count, inst, max_iter, bp) != FFCZ_OK) return 0;
  g_err = keep;
  return bp.bytes;
}

int32_t ffcz_correct_batched(int32_t dtype, int32_t count, const ffcz_instance* inst, int32_t max_iter,
                             const ffcz_options* opts, void* ws, size_t ws_bytes, void* stream, ffcz_stats* stats) {
  if (max_iter < 0) return fail(FFCZ_E_INVALID, "max_iter must be >= 0");
  BatchPlan bp;
  int32_t r = batch_plan(dtype, count, inst, max_iter, bp);
  if (r != FFCZ_OK) return r;
  if (!ws || ws_bytes < bp.bytes || ((uintptr_t)ws & 255))
    return fail(FFCZ_E_WORKSPACE, "workspace smaller than ffcz_batched_workspace_bytes() or misaligned");
  ffcz_options o;
  if (opts) o = *opts;
  else ffcz_default_options(&o);
  o.masks_out = nullptr;
  o.viol_per_round = nullptr;
  for (int i = 0; i < count; ++i) {
    const ffcz_instance& in = inst[i];
    if (!in.x_orig || !in.x_base || !in.x_out) return fail(FFCZ_E_INVALID, "null data pointer");
    if (in.x_orig == in.x_base || in.x_orig == in.x_out) return fail(FFCZ_E_INVALID, "x_orig must not alias");
    if (!std::isfinite(in.eps_s) || in.eps_s < 0 || !std::isfinite(in.delta_f) || in.delta_f < 0)
      return fail(FFCZ_E_INVALID, "bounds must be finite and >= 0");
    if (((uintptr_t)in.x_orig & 15) || ((uintptr_t)in.x_base & 15) || ((uintptr_t)in.x_out & 15))
      return fail(FFCZ_E_WORKSPACE, "data must be 16-byte aligned");
  }
  hipStream_t s = (hipStream_t)stream;
  char* w = (char*)ws;
  // margins: per instance (FP32: suggested from x, all members in one launch; FP64: 2^-16).  The
  // thresholds of 1D members are set on the device; a batch without groups reads the margins
  // back with the statistics.
  const bool derive = !(o.margin_rel > 0.0) && dtype == FFCZ_F32 && count > 0;
  std::vector<double> mus(count, o.margin_rel > 0.0 ? o.margin_rel : std::ldexp(1.0, -16));
  double* const dmu = (double*)(w + bp.off_msum) + (size_t)count * kUlpSlots;
  std::map<int, int> first;
  if (count > 0) {
    r = sig_stage(bp, count, inst, derive ? nullptr : mus.data(), w, s, g_host_sig, first);
    if (r != FFCZ_OK) return r;
  }
  if (derive) {
    int64_t nmax = 1;
    for (int i = 0; i < count; ++i) nmax = std::max(nmax, ((const MarginJob*)g_host_sig.p)[i].n);
    const MarginJob* dj = (const MarginJob*)(w + bp.off_mjobs);
    double* dpart = (double*)(w + bp.off_msum);
    const unsigned bx = (unsigned)ulp_slots(nmax);
    for (int c0 = 0; c0 < count; c0 += 65535) {  // grid y holds at most 65535 fields
      const int nc = std::min(65535, count - c0);
      hipLaunchKernelGGL(ulp_part_kernel, dim3(bx, (unsigned)nc), dim3(256), 0, s, MarginJob{}, dj + c0,
                         dpart + (size_t)c0 * kUlpSlots);
      HIPCHK(hipGetLastError());
    }
    hipLaunchKernelGGL(margin_kernel, dim3((unsigned)count), dim3(256), 0, s, (const double*)dpart, MarginJob{}, dj,
                       (int)FFCZ_F32, dmu, (DevState*)nullptr, (SigDesc*)(w + bp.off_desc));
    HIPCHK(hipGetLastError());
    if (!bp.groups.empty()) {
      HIPCHK(g_host_misc.reserve(sizeof(double) * count));
      HIPCHK(hipMemcpyAsync(g_host_misc.p, dmu, sizeof(double) * count, hipMemcpyDeviceToHost, s));
      HIPCHK(hipStreamSynchronize(s));
      memcpy(mus.data(), g_host_misc.p, sizeof(double) * count);
    }
  }
  r = sig_tables(bp, w, s);
  if (r != FFCZ_OK) return r;
  std::vector<int32_t> status(count, FFCZ_OK);
  if (!bp.sig_ids.empty() && !bp.groups.empty()) {
    r = dtype == FFCZ_F32 ? mixed_batch<float>(bp, inst, mus, max_iter, o, w, s, first, stats, status)
                          : mixed_batch<double>(bp, inst, mus, max_iter, o, w, s, first, stats, status);
    if (r != FFCZ_OK) return r;
  } else {
    r = pretune_sigs(bp, o, w, s, first);
    if (r != FFCZ_OK) return r;
    r = run_sigs(bp, max_iter, o, w, s, first, g_host_sigstate);
    if (r != FFCZ_OK) return r;
    for (size_t g = 0; g < bp.groups.size(); ++g) {
      const Plan& p = bp.gplans[g];
      std::vector<ffcz_instance> gi;
      std::vector<double> gm;
      for (int id : bp.groups[g]) {
        gi.push_back(inst[id]);
        gm.push_back(mus[id]);
      }
      std::vector<int32_t> gs(gi.size(), FFCZ_OK);
      std::vector<ffcz_stats> gst(gi.size());
      r = dtype == FFCZ_F32
              ? correct_group<float>(p, gi.data(), gm.data(), max_iter, o, w + bp.goff[g], s, gst.data(), gs.data())
              : correct_group<double>(p, gi.data(), gm.data(), max_iter, o, w + bp.goff[g], s, gst.data(), gs.data());
      if (r != FFCZ_OK) return r;
      for (size_t k = 0; k < gi.size(); ++k) {
        status[bp.groups[g][k]] = gs[k];
        if (stats) stats[bp.groups[g][k]] = gst[k];
      }
    }
  }
  r = collect_sigs(bp, inst, mus, derive && bp.groups.empty() ? dmu : nullptr, o, w, s, stats, status.data());
  if (r != FFCZ_OK) return r;
  if (stats)
    for (int i = 0; i < count; ++i) stats[i].status = status[i];
  const int32_t wst = worst(status);
  if (wst == FFCZ_VERIFY_FAILED) g_err = "FP64 re-verification failed for at least one instance";
  return wst;
}

int32_t ffcz_correct_backward(int32_t dtype, int32_t ndim, const int64_t* shape, int32_t rounds, const void* masks,
                              const void* gy, void* gb, void* ws, size_t ws_bytes, void* stream) {
  if (route_1d(ndim, shape)) return fail(FFCZ_E_SHAPE, "the adjoint needs a power-of-two field (masks are recorded there)");
  Plan p;
  int32_t r = make_plan(dtype, ndim, shape, rounds, 1, p);
  if (r != FFCZ_OK) return r;
  if (!masks || !gy || !gb) return fail(FFCZ_E_INVALID, "null pointer");
  if (((uintptr_t)gy & 15) || ((uintptr_t)gb & 15)) return fail(FFCZ_E_WORKSPACE, "gradients must be 16-byte aligned");
  if (!ws || ws_bytes < p.bytes) return fail(FFCZ_E_WORKSPACE, "workspace smaller than ffcz_workspace_bytes()");
  if ((uintptr_t)ws & 255) return fail(FFCZ_E_WORKSPACE, "workspace must be 256-byte aligned");
  hipStream_t s = (hipStream_t)stream;
  // the last-axis plan the table holds for this geometry (no timing here): the adjoint's
  // last-axis passes take the direct form where the forward loop pass does
  if (p.H >= 64) {
    int vz = 0;
    r = tune_pass(tune_key_z(p), s, false, 0.98f, kRowVariants, [](int) { return hipSuccess; }, &vz);
    if (r != FFCZ_OK) return r;
    set_variants(p, 0, 0, masked_variant(p, vz));
  }
  if (dtype == FFCZ_F32) return backward_impl<float>(p, rounds, masks, gy, gb, ws, s);
  return backward_impl<double>(p, rounds, masks, gy, gb, ws, s);
}

}  // extern "C"
