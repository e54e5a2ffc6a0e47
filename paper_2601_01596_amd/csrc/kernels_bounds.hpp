// Set-up kernels of the generalised bounds (the footnote to Eq. 2 in Sec. IV-A; Sec. V-B,
// Observation 4): pointwise spectral bounds copied into the spectrum layout, their checks and
// minimum, and the pointwise bound that keeps every shell of the power spectrum within a
// relative error.
//
// Power-spectrum bound.  Shell b = rint(|k|) (|k| from the signed integer frequencies) holds
// P_b = sum w_k |X_k|^2 with full-spectrum weights w_k (2 for interior last-axis entries, 1 at
// k_z = 0 and at the Nyquist plane).  For an error with |Re|, |Im| <= D on every entry of the
// shell (box), |P_hat_b - P_b| <= 2 sqrt2 D S_b + 2 D^2 W_b with S_b = sum w_k |X_k| and
// W_b = sum w_k; for |delta_k| <= D (disk) it is at most 2 D S_b + D^2 W_b.  D_b is the
// positive root of that bound = rho P_b, computed as rho P_b / (sqrt(2 S^2 + 2 W rho P) +
// sqrt2 S) (box) or rho P_b / (sqrt(S^2 + W rho P) + S) (disk), which has no cancellation.
#pragma once
#include "common.hpp"

namespace ffcz {

constexpr int kMaxShells = 2560;  // rint(|k|) + 1 for every supported shape (at most 2,509)
constexpr int kMinSlots = 1024;   // block minima of a bound set

// Geometry of a half-spectrum laid out in rows of ncols entries, rows grouped in planes of
// 2^lg_rpp rows at a pitch / plane stride (complex entries).
struct SpecGeom {
  int64_t nrows;
  int32_t ncols, lg_rpp;
  int64_t pitch, plane;
};

// Entries e0, e0 + step, ... of a half-spectrum as (row, column), without a division per entry.
struct EntryWalk {
  int32_t ncols, dr, dk, r, k;
  __device__ __forceinline__ EntryWalk(int64_t e0, int64_t step, int32_t nc) : ncols(nc) {
    r = (int32_t)(e0 / nc);
    k = (int32_t)(e0 - (int64_t)r * nc);
    dr = (int32_t)(step / nc);
    dk = (int32_t)(step - (int64_t)dr * nc);
  }
  __device__ __forceinline__ void next() {
    r += dr;
    k += dk;
    if (k >= ncols) {
      k -= ncols;
      ++r;
    }
  }
};

// Shell rint(|k|) of an entry: |k|^2 is an integer below 2^24 (extents of at most 4096), exact
// in FP32, and shell b holds the integers b (b - 1) + 1 ... b (b + 1), so an FP32 square root
// put right by one step gives the shell without FP64 work.
__device__ __forceinline__ int shell_of(int k2) {
  int b = (int)rintf(sqrtf((float)k2));
  b += k2 > b * b + b ? 1 : 0;
  b -= (b > 0 && k2 <= b * b - b) ? 1 : 0;
  return b;
}
// |k|^2 of entry (r, kz): r = i0 (2D) or i0 n1 + i1 (3D; n1 = 2^lg1), signed frequencies.
__device__ __forceinline__ int entry_k2(int nd, int r, int kz, int n0, int lg1) {
  auto sfreq = [](int k, int n) -> int { return k < (n + 1) / 2 ? k : k - n; };
  int k2 = kz * kz;
  if (nd == 3) {
    const int f0 = sfreq(r >> lg1, n0), f1 = sfreq(r & ((1 << lg1) - 1), 1 << lg1);
    k2 += f0 * f0 + f1 * f1;
  } else if (nd == 2) {
    const int f0 = sfreq(r, n0);
    k2 += f0 * f0;
  }
  return k2;
}

// Bits of a non-negative double (they order as integers).
__device__ __forceinline__ unsigned long long dbits(double v) { return (unsigned long long)__double_as_longlong(v); }

// The caller's spectral bounds (M entries in C order, or scalars when the arrays are null) as
// (Re, Im) pairs in the working type at the spectrum's layout.  A scalar is rounded toward zero
// in FP32 (the bound does not grow); arrays arrive in the working type.  bad counts entries
// that are negative or not finite; minpart[block] receives the block's smallest bound.  Bound by
// the copy (256^3 FP32 31 -> 28 us; one entry a lane with a division each before).
template <typename T>
__global__ void __launch_bounds__(256) bounds_setup_kernel(const T* dre, const T* dim, double sre, double sim,
                                                           cx<T>* out, int64_t M, SpecGeom g,
                                                           unsigned long long* minpart, unsigned long long* bad) {
  __shared__ unsigned long long red[4];
  unsigned long long nbad = 0;
  const T inf = (T)__builtin_huge_val();
  T mn = inf;
  const T cre = to_t<T>(sre), cim = to_t<T>(sim);
  // two entries a lane, so that a row's stores are 16 bytes wide (FP32) and cover its last line:
  // entry ncols of a row with an odd count is padding (pitch is even), stored as zero
  const int npr = (g.ncols + 1) / 2, rpm = (1 << g.lg_rpp) - 1;
  const int64_t np = g.nrows * npr, step = (int64_t)gridDim.x * 256;
  const int64_t f0 = (int64_t)blockIdx.x * 256 + threadIdx.x;
  EntryWalk w(f0, step, npr);
  auto check = [&](T br, T bi) {
    const bool ok = isfinite(br) && isfinite(bi) && br >= T(0) && bi >= T(0);
    nbad += ok ? 0 : 1;
    const T m = (br < bi ? br : bi) + T(0);  // -0 to 0: its bits would order above every bound
    if (ok) mn = mn < m ? mn : m;
  };
  struct alignas(2 * sizeof(cx<T>) < 16 ? 16 : 2 * sizeof(cx<T>)) Pair {
    cx<T> a, b;
  };
#pragma unroll 2
  for (int64_t f = f0; f < np; f += step, w.next()) {
    const int k = 2 * w.k;
    const bool two = k + 1 < g.ncols;
    const int64_t e = (int64_t)w.r * g.ncols + k, e1 = two ? e + 1 : e;
    const T r0 = dre ? dre[e] : cre, r1 = dre ? dre[e1] : cre;
    const T i0 = dim ? dim[e] : (dre ? r0 : cim), i1 = dim ? dim[e1] : (dre ? r1 : cim);
    check(r0, i0);
    if (two) check(r1, i1);
    Pair q{{r0, i0}, {two ? r1 : T(0), two ? i1 : T(0)}};
    *reinterpret_cast<Pair*>(out + (int64_t)(w.r >> g.lg_rpp) * g.plane + (int64_t)(w.r & rpm) * g.pitch + k) = q;
  }
  unsigned long long mb = mn == inf ? ~0ull : dbits((double)mn);
  for (int off = 32; off > 0; off >>= 1) {
    const unsigned long long o = __shfl_xor(mb, off, 64);
    mb = mb < o ? mb : o;
    nbad += __shfl_xor(nbad, off, 64);
  }
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = mb;
  if ((threadIdx.x & 63) == 0 && nbad) atomicAdd(bad, nbad);
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long m = red[0];
    for (int w = 1; w < 4; ++w) m = m < red[w] ? m : red[w];
    minpart[blockIdx.x] = m;
  }
}

// Spatial bounds E_n: count entries that are negative or not finite.
template <typename T>
__global__ void __launch_bounds__(256) spatial_check_kernel(const T* E, int64_t n, unsigned long long* bad) {
  unsigned long long nbad = 0;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    const double v = (double)E[i];
    nbad += (isfinite(v) && v >= 0.0) ? 0 : 1;
  }
  for (int off = 32; off > 0; off >>= 1) nbad += __shfl_xor(nbad, off, 64);
  if ((threadIdx.x & 63) == 0 && nbad) atomicAdd(bad, nbad);
}

// Per-shell sums of the FP64 spectrum W of x: each block adds its entries into LDS shells
// (atomic adds, so the order of the additions is not fixed), then stores its partial sums
// part[block][3][nb] (P, S, W).  Reading W bounds it; 16 waves a CU and four entries a lane in
// flight, integer shells and counts: 256^3 90 -> 36 us, 3.8 TB/s (4 waves, FP64 shells and counts before).
constexpr int kShellLanes = 1024;
__global__ void __launch_bounds__(kShellLanes) shell_part_kernel(const cx<double>* W, SpecGeom g, int nd, int n0,
                                                                 int lg1, int nl, int nb, double* part) {
  __shared__ double sh[2 * kMaxShells];
  __shared__ uint32_t shw[kMaxShells];
  constexpr int NT = kShellLanes, U = 4;
  for (int i = threadIdx.x; i < 2 * nb; i += NT) sh[i] = 0.0;
  for (int i = threadIdx.x; i < nb; i += NT) shw[i] = 0u;
  __syncthreads();
  const int64_t M = g.nrows * g.ncols, step = (int64_t)gridDim.x * NT;
  int64_t e = (int64_t)blockIdx.x * NT + threadIdx.x;
  EntryWalk w(e, step, g.ncols);
  const int rpm = (1 << g.lg_rpp) - 1;
  while (e < M) {
    cx<double> X[U];
    int b[U];
    uint32_t wt[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      wt[u] = 0u;
      if (e < M) {
        X[u] = W[(int64_t)(w.r >> g.lg_rpp) * g.plane + (int64_t)(w.r & rpm) * g.pitch + w.k];
        b[u] = shell_of(entry_k2(nd, w.r, w.k, n0, lg1));
        wt[u] = (w.k == 0 || 2 * w.k == nl) ? 1u : 2u;
      }
      e += step;
      w.next();
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (wt[u]) {
        const double wd = (double)wt[u], a2 = X[u].re * X[u].re + X[u].im * X[u].im;
        atomicAdd(&sh[b[u]], wd * a2);
        atomicAdd(&sh[nb + b[u]], wd * sqrt(a2));
        atomicAdd(&shw[b[u]], wt[u]);
      }
    }
  }
  __syncthreads();
  double* out = part + (int64_t)blockIdx.x * 3 * nb;
  for (int i = threadIdx.x; i < 2 * nb; i += NT) out[i] = sh[i];
  for (int i = threadIdx.x; i < nb; i += NT) out[2 * nb + i] = (double)shw[i];
}

// Add the block partials (64 slices of blocks side by side, then the slices in order) and take
// D_b.  A block does 16 shells: one 128-byte line of each partial row.  One lane a shell, the
// blocks in a row, took 73 us at 222 shells and 256 blocks, the latency of 256 loads; 5 us now.
__global__ void __launch_bounds__(1024) shell_bound_kernel(const double* part, int nblk, int nb, double rho,
                                                           int disk, double* bins) {
  __shared__ double red[3][64][17];
  const int c = threadIdx.x & 15, sl = threadIdx.x >> 4;
  const int b = blockIdx.x * 16 + c;
  double v[3] = {0.0, 0.0, 0.0};
  if (b < nb)
    for (int k = sl; k < nblk; k += 64) {
      const double* q = part + (int64_t)k * 3 * nb + b;
#pragma unroll
      for (int i = 0; i < 3; ++i) v[i] += q[i * nb];
    }
#pragma unroll
  for (int i = 0; i < 3; ++i) red[i][sl][c] = v[i];
  __syncthreads();
  if (sl != 0 || b >= nb) return;
  for (int k = 1; k < 64; ++k)
#pragma unroll
    for (int i = 0; i < 3; ++i) v[i] += red[i][k][c];
  const double P = v[0], S = v[1], Wt = v[2];
  const double den = disk ? sqrt(S * S + Wt * rho * P) + S : sqrt(2.0 * S * S + 2.0 * Wt * rho * P) + sqrt(2.0) * S;
  bins[b] = den > 0.0 ? rho * P / den : 0.0;
}

// The shell bound of every half-spectrum entry, in C order, in the field's dtype (rounded
// toward zero in FP32: the bound does not grow).  256^3 34 -> 22 us with integer shells.
template <typename T>
__global__ void __launch_bounds__(256) shell_scatter_kernel(const double* bins, int64_t nrows, int32_t ncols, int nd,
                                                            int n0, int lg1, T* out) {
  const int64_t M = nrows * ncols, step = (int64_t)gridDim.x * 256;
  const int64_t e0 = (int64_t)blockIdx.x * 256 + threadIdx.x;
  EntryWalk w(e0, step, ncols);
  constexpr int U = 4;
  for (int64_t e = e0; e < M;) {
    double d[U];
#pragma unroll
    for (int u = 0; u < U; ++u, w.next()) d[u] = bins[e + u * step < M ? shell_of(entry_k2(nd, w.r, w.k, n0, lg1)) : 0];
#pragma unroll
    for (int u = 0; u < U; ++u, e += step)
      if (e < M) out[e] = to_t<T>(d[u]);
  }
}

}  // namespace ffcz
