// The loop's y-inverse, last-axis and y-forward passes of a 3D field as one pass, for planes
// (one x index: n1 rows of the half spectrum) that fit in one block's LDS.
//
// Separately, the three passes of a small field are three launches of a few microseconds each
// that move the spectrum three times through the caches; what bounds them is launch, fill and
// latency, not bandwidth.  Here a block reads its plane once after the x-pass, keeps it in LDS
// through
//     inverse along y (in place, column groups), C2R, s-clip, R2C (rows), forward along y
// and stores it twice: the last-axis R2C (Z, the iterate a closing pass starts from) and its
// y-forward transform (A, which the next x-pass reads).  It begins with the round's check.  5 M c
// bytes a round instead of 8 M c, and two launches (x-pass, plane) instead of five.  Each transform runs on the stage
// plan and with the formulas of the separate passes.
//
// Lanes: columns fastest in the y transforms (groups of CG columns, as many as the block's lanes
// hold), rows fastest in the last-axis ones; the odd row pitch H + 1 keeps both on distinct
// banks.  Lanes past a group's last item repeat another lane's work (same values to the same
// slots) and store and count nothing, so that every lane meets every barrier.
#pragma once
#include "kernels_ctl.hpp"

namespace ffcz {

template <typename T>
struct PlaneArgs {
  cx<T>* A;             // in: after the x-pass; out: y-forward transform of the new iterate
  cx<T>* Z;             // out: last-axis R2C of the new iterate
  int64_t pitch, plane; // complex entries per row / per plane
  int64_t nplanes;      // planes per instance
  const cx<T>* twy;     // stage twiddles of the y length
  const cx<T>* twz;     // stage twiddles of length H, then the H R2C twiddles
  DevState* st;
  unsigned long long* part;  // s-clip count of each plane
  // the check the pass starts with: violation counts of the x-pass (nx an instance), clip counts
  // of the checked iterate (nz an instance)
  const unsigned long long* xpart;
  const unsigned long long* zpart;
  int64_t nx, nz;
  int32_t round, pad;
  unsigned long long* viol;
  int64_t vstride;
  Post post;
};

// Lane plan of one (type, y length, H).
template <int LY, int H>
struct PlaneGeom {
  static constexpr int EY = pick_E(LY), PY = LY / EY;
  static constexpr int EZ = pick_E_row(H), PZ = H / EZ;
  static constexpr int NC = H + 1, PT = H + 1;
  static constexpr int CMAX = 1024 / PY;               // columns 1024 lanes hold
  static constexpr int NG = (NC + CMAX - 1) / CMAX;    // column groups
  static constexpr int CG = (NC + NG - 1) / NG;        // columns per group
  static constexpr int NCL = CG * PY;                  // lanes with a column
  static constexpr int NT0 = (NCL + 63) / 64 * 64;
  static constexpr int NT = NT0 < PZ ? PZ : NT0;
  static constexpr int rg() {
    int r = 1;
    while (r < LY && 2 * r * PZ <= NT) r *= 2;
    return r;
  }
  static constexpr int RG = rg(), NR = LY / RG, NRL = RG * PZ;  // rows per group, groups, lanes with a row
  static constexpr int TWY = Sched<LY, EY>::twsize, TWZ = Sched<H, EZ>::twsize;
};

// Entries (y length x H) up to which a plane fits in LDS beside the twiddle tables, per type.
constexpr int kPlaneMinLy = 16, kPlaneMaxLy = 512, kPlaneMinH = 8, kPlaneMaxH = 256;
template <typename T>
__host__ __device__ constexpr bool plane_fits(int LY, int H) {
  return LY >= kPlaneMinLy && LY <= kPlaneMaxLy && H >= kPlaneMinH && H <= kPlaneMaxH &&
         (int64_t)LY * H * (int64_t)sizeof(cx<T>) <= 128 * 1024;
}

template <typename T, int LY, int H>
__global__ void __launch_bounds__((PlaneGeom<LY, H>::NT)) plane_kernel(PlaneArgs<T> a) {
  using G = PlaneGeom<LY, H>;
  constexpr int EY = G::EY, PY = G::PY, EZ = G::EZ, PZ = G::PZ, PT = G::PT, NT = G::NT;
  constexpr int NW = NT / 64 > 0 ? (NT + 63) / 64 : 1;
  __shared__ cx<T> pl[LY * PT];
  __shared__ cx<T> twy[G::TWY > 0 ? G::TWY : 1];
  __shared__ cx<T> twz[G::TWZ + H];
  __shared__ unsigned long long red[NW], redz[NW];
  __shared__ int32_t done;

  const int64_t o = blockIdx.x;
  const int64_t inst = o / a.nplanes;
  DevState* st = a.st + inst;
  const int t = threadIdx.x;
  for (int i = t; i < G::TWY; i += NT) twy[i] = a.twy[i];
  for (int i = t; i < G::TWZ + H; i += NT) twz[i] = a.twz[i];
  const cx<T>* rtw = twz + G::TWZ;
  cx<T>* const gA = a.A + o * a.plane;
  cx<T>* const gZ = a.Z + o * a.plane;

  const int tc = t % G::NCL;  // column mapping
  const int cl = tc % G::CG, jc = tc / G::CG;
  const int tr = t % G::NRL;  // row mapping
  const int rl = tr % G::RG, jr = tr / G::RG;

  // ---- the check: every block sums the x-pass counts and comes to the same decision; the block
  // of the first plane records it.  The done flag is read by one lane for the whole block: the
  // first plane's block may set it while this one starts (a stop, which this block then either
  // sees in the flag or decides itself), and waves that read it at different times would part.
  const T sc = (T)st->inv_n;
  const T Ep = to_t<T>(st->Ep);
  auto col_of = [&](int g) { return g * G::CG + cl < H ? g * G::CG + cl : H; };
  auto load_cols = [&](cx<T> (&v)[EY], int g) {
    const cx<T>* src = gA + (int64_t)jc * a.pitch + col_of(g);
#pragma unroll
    for (int q = 0; q < EY; ++q) v[q] = src[(int64_t)(q * PY) * a.pitch];
  };
  cx<T> vy[EY];
  load_cols(vy, 0);  // in flight across the check
  {
    unsigned long long sx = 0, sz = 0;
    for (int64_t i = t; i < a.nx; i += NT) sx += a.xpart[inst * a.nx + i];
    const bool rec = o == inst * a.nplanes;
    if (rec)
      for (int64_t i = t; i < a.nz; i += NT) sz += a.zpart[inst * a.nz + i];
    sx = wave_sum_u64(sx);
    sz = wave_sum_u64(sz);
    if (t == 0) done = *(volatile int32_t*)&st->done;
    if ((t & 63) == 0) {
      red[t >> 6] = sx;
      redz[t >> 6] = sz;
    }
    __syncthreads();
    if (done) return;
    sx = 0;
    for (int w = 0; w < NW; ++w) sx += red[w];
    const bool stop = check_stops(st, a.round, sx);
    if (rec && t == 0) {
      sz = 0;
      for (int w = 0; w < NW; ++w) sz += redz[w];
      record_check(st, a.round, sx, sz, stop, a.viol + inst * a.vstride, a.post, inst);
    }
    if (stop) return;
  }

  // ---- inverse along y: global -> registers -> plane
#pragma unroll 1
  for (int g = 0; g < G::NG; ++g) {
    const int c = col_of(g);
    fft<T, LY, EY, true, PT, 1>(vy, pl, twy, c, jc);
    if constexpr (Sched<LY, EY>::nst > 1) __syncthreads();
#pragma unroll
    for (int q = 0; q < EY; ++q) pl[(jc + q * PY) * PT + c] = vy[q];
    if (g + 1 < G::NG) load_cols(vy, g + 1);
  }
  __syncthreads();

  // ---- rows: C2R, 1/N, s-clip, forward transform
  uint32_t cnt = 0;
#pragma unroll 1
  for (int g = 0; g < G::NR; ++g) {
    const int row = g * G::RG + rl;
    cx<T>* const lrow = pl + row * PT;
    cx<T> v[EZ];
#pragma unroll
    for (int q = 0; q < EZ; ++q) {
      const int k = jr + q * PZ;
      cx<T> A = lrow[k];
      cx<T> B = lrow[H - k];
      if (k == 0) {
        A.im = T(0);
        B.im = T(0);
      }
      const cx<T> sm = A + conjg(B);
      const cx<T> df = cmulc(A - conjg(B), rtw[k]);  // W^-k (A - B*)
      v[q] = cx<T>{sm.re - df.im, sm.im + df.re};    // sm + i * df
    }
    fft<T, H, EZ, true, 1, PT>(v, pl, twz, row, jr);
#pragma unroll
    for (int q = 0; q < EZ; ++q) {
      const T e0 = v[q].re * sc, e1 = v[q].im * sc;
      const bool k0 = fabs(e0) <= Ep, k1 = fabs(e1) <= Ep;
      cnt += (!k0) + (!k1);
      v[q] = cx<T>{clipv(e0, Ep), clipv(e1, Ep)};
    }
    fft<T, H, EZ, false, 1, PT>(v, pl, twz, row, jr);
    __syncthreads();
#pragma unroll
    for (int q = 0; q < EZ; ++q) lrow[jr + q * PZ] = v[q];
  }
  if (t >= G::NRL) cnt = 0;
  __syncthreads();

  // ---- R2C in place: a lane owns entries k and H - k of a row
  constexpr int HP = H / 2 + 1;
  for (int f = t; f < LY * HP; f += NT) {
    const int r = f / HP, k = f - r * HP;
    cx<T>* const zr = pl + r * PT;
    const cx<T> Zk = zr[k];
    const cx<T> Zm = zr[(H - k) & (H - 1)];
    auto unpack = [&](cx<T> P, cx<T> Q, int i) -> cx<T> {
      const cx<T> ev = scal(P + conjg(Q), T(0.5));
      const cx<T> d = P - conjg(Q);
      const cx<T> od = cx<T>{d.im * T(0.5), -d.re * T(0.5)};  // d / (2i)
      return ev + cmul(rtw[i], od);
    };
    zr[k] = unpack(Zk, Zm, k);
    if (k == 0) zr[H] = cx<T>{Zk.re - Zk.im, T(0)};
    else if (2 * k < H) zr[H - k] = unpack(Zm, Zk, H - k);
  }
  __syncthreads();

  // ---- Z, and the forward transform along y to A
#pragma unroll 1
  for (int g = 0; g < G::NG; ++g) {
    const int c0 = g * G::CG + cl;
    const int c = c0 < H ? c0 : H;
    const bool own = t < G::NCL && c0 <= H;
    cx<T> v[EY];
#pragma unroll
    for (int q = 0; q < EY; ++q) {
      v[q] = pl[(jc + q * PY) * PT + c];
      if (own) gZ[(int64_t)(jc + q * PY) * a.pitch + c] = v[q];
    }
    fft<T, LY, EY, false, PT, 1>(v, pl, twy, c, jc);
    if (own) {
#pragma unroll
      for (int q = 0; q < EY; ++q) gA[(int64_t)(jc + q * PY) * a.pitch + c] = v[q];
    }
  }

  unsigned long long s = wave_sum_u64(cnt);
  if ((t & 63) == 0) red[t >> 6] = s;
  __syncthreads();
  if (t == 0) {
    s = 0;
    for (int w = 0; w < NW; ++w) s += red[w];
    a.part[o] = s;
  }
}

}  // namespace ffcz
