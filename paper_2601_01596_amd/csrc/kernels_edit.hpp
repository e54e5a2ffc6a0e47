// Edit coding around the correction loop (Alg. 1 edit bookkeeping, CompactEdits and
// QuantizeEdits of Sec. IV-B / IV-D, and their inverse for applying edits).
//
// Coordinates.  The spatial edits have one coordinate per real point (C order).
// The frequency edits have two per half-spectrum entry, Re then Im, entries in C
// order over rows of H + 1 entries; in the workspace those rows sit at the
// spectrum's padded pitch and plane.  A flag bit per coordinate says whether its
// edit is non-zero; flags are packed eight to a byte, coordinate 8 b + i in bit i
// of byte b (least significant bit first).  The non-zero edits are stored in
// coordinate order, each at the exclusive prefix count of the flags before it,
// as m-bit quantisation codes rint(v / step) (int32, half to even).
//
// Work split.  A wave takes 64 consecutive coordinates at a time (one lane each),
// so its ballot IS the 64-bit flag word of those coordinates, and mbcnt of the
// ballot is each lane's prefix inside the word.  A block owns kEditChunks
// consecutive words, wave w a run of kEditWords of them.  Three launches, each over
// both sets: the first reads every value once, writes the flag words and counts each
// block's, a scan turns the counts into block offsets (a block per set), the third
// reads the flag words and, at flagged coordinates only, the values, and writes the
// codes.  The decoder counts the given flag words, scans, and expands.  Reading the
// values bounds the first, storing them the last; a wave keeps kEditBatch loads in
// flight and walks rows without divisions.  256^3 FP32, both sets: count 57 -> 25 us (5.4 TB/s),
// scan 22 -> 4, write 77 -> 29, flag count 31 -> 6, expand 78 -> 33 (4 TB/s; one
// launch per set and a barrier per four words before).
#pragma once
#include <type_traits>

#include "common.hpp"

namespace ffcz {

constexpr int kEditWaves = 4;                     // waves per block (256 lanes)
constexpr int kEditWords = 16;                    // 64-coordinate words per wave
constexpr int kEditBatch = 8;                     // words of a wave in flight
constexpr int kEditChunks = kEditWaves * kEditWords;  // words per block
constexpr int64_t kEditBlockCoords = 64 * kEditChunks;

// One coordinate set: the spatial edits (dense, C order) or the frequency edits
// (complex entries in the padded spectrum layout, Re/Im interleaved).
template <typename T>
struct EditSet {
  T* val;           // spatial: N values; frequency: the spectrum buffer as reals
  int64_t ncoord;   // N, or 2 M
  int32_t freq;     // 0 spatial, 1 frequency
  int32_t ncols;    // frequency: entries per row (H + 1)
  int64_t pitch;    // frequency: complex entries per row of the buffer
  int64_t plane;    // frequency: complex entries per plane of 2^lg_rpp rows
  int32_t lg_rpp;
  int32_t pad;
  double inv;       // frequency: 1 / ncols
};

// Element offset (in T) of coordinate c of a set.
template <typename T>
__device__ __forceinline__ int64_t edit_offset(const EditSet<T>& s, int64_t c) {
  if (!s.freq) return c;
  const int64_t e = c >> 1;
  const int64_t r = e / s.ncols;
  const int64_t col = e - r * s.ncols;
  const int64_t addr = (r >> s.lg_rpp) * s.plane + (r & ((int64_t(1) << s.lg_rpp) - 1)) * s.pitch + col;
  return 2 * addr + (c & 1);
}

__device__ __forceinline__ int lane_prefix(unsigned long long m) {
  // set bits of m below this lane
  return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Offsets of a lane's coordinates c, c + 64, c + 128, ... of a wave's run, relative to an element
// all its lanes share (`base`), in bytes and 32 bits.  K 0: dense.  K 1: rows of at least 32 entries, so that
// 64 coordinates (32 entries) cross at most one row end, by selects and additions.  K 2: shorter
// rows, by division.  (The address arithmetic bounds these kernels, not their loads.)
template <typename T, int K>
struct CoordWalk {
  const EditSet<T>& s;
  int64_t base;
  uint32_t off;  // bytes of this lane's coordinate from base
  int32_t r = 0, col = 0, rmask = 0;
  uint32_t row_pad = 0, plane_pad = 0;
  int64_t e = 0;
  __device__ __forceinline__ CoordWalk(const EditSet<T>& set, int64_t c0, int lane) : s(set), base(c0), off(lane * (uint32_t)sizeof(T)) {
    if constexpr (K > 0) {
      const int64_t e0 = c0 >> 1;  // c0 is a multiple of 64
      rmask = (1 << s.lg_rpp) - 1;
      if constexpr (K == 1) {
        // row of e0 from the reciprocal, put right by one
        int64_t r0 = (int64_t)((double)e0 * s.inv);
        int64_t k0 = e0 - r0 * s.ncols;
        if (k0 < 0) {
          --r0;
          k0 += s.ncols;
        } else if (k0 >= s.ncols) {
          ++r0;
          k0 -= s.ncols;
        }
        row_pad = (uint32_t)(2 * (s.pitch - s.ncols) * (int64_t)sizeof(T));
        plane_pad = (uint32_t)(2 * (s.plane - (s.pitch << s.lg_rpp)) * (int64_t)sizeof(T));
        base = at(r0, k0);
        // one value for the wave (in scalar registers)
        base = (int64_t)((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)base) |
                         (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(base >> 32)) << 32);
        r = (int32_t)(r0 & rmask);
        col = (int32_t)k0;
        move(lane >> 1);
      } else {
        e = e0 + (lane >> 1);
        place(lane);
      }
    }
  }
  __device__ __forceinline__ int64_t at(int64_t row, int64_t k) const {
    return 2 * ((row >> s.lg_rpp) * s.plane + (row & rmask) * s.pitch + k);
  }
  // n <= 31 or 32 entries on, past at most one row end (off already counts them)
  __device__ __forceinline__ void move(int n) {
    col += n;
    const bool wrap = col >= s.ncols;
    col -= wrap ? s.ncols : 0;
    off += wrap ? row_pad : 0;
    const bool turn = wrap && r == rmask;  // the last row of a plane
    off += turn ? plane_pad : 0;
    r = wrap ? (turn ? 0 : r + 1) : r;
  }
  __device__ __forceinline__ void place(int lane) {
    const int64_t row = e / s.ncols;
    base = at(row, e - row * s.ncols);
    off = (lane & 1) * (uint32_t)sizeof(T);
  }
  __device__ __forceinline__ void next(int lane) {
    if constexpr (K == 2) {
      e += 32;
      place(lane);
    } else {
      off += 64 * (uint32_t)sizeof(T);
      if constexpr (K == 1) move(32);
    }
  }
  __device__ __forceinline__ T* ptr() const {
    return reinterpret_cast<T*>(reinterpret_cast<char*>(s.val + base) + off);
  }
};

// One coordinate set of a coding or expanding call.
template <typename T>
struct EditJob {
  EditSet<T> s;
  int64_t nb;               // blocks
  unsigned long long* off;  // per block: count, then exclusive offset
  unsigned long long* total;
  uint8_t* flags;
  int32_t* codes;
  int64_t ncodes;  // decoder: codes given
  double step;
};

// A wave's kEditWords flag words, lane i < kEditWords holding word i (bits past the last
// coordinate zero), in the flag bytes from word w0 on.
__device__ __forceinline__ unsigned long long load_words(const uint8_t* flags, int64_t ncoord, int64_t w0, int lane) {
  const int64_t nbytes = (ncoord + 7) >> 3, i = w0 + lane;
  if (lane >= kEditWords || i * 64 >= ncoord) return 0ull;
  unsigned long long m = 0;
  if (i * 8 + 8 <= nbytes) m = *reinterpret_cast<const unsigned long long*>(flags + i * 8);
  else
    for (int k = 0; i * 8 + k < nbytes; ++k) m |= (unsigned long long)flags[i * 8 + k] << (8 * k);
  const int64_t rem = ncoord - i * 64;
  return rem < 64 ? m & ((1ull << rem) - 1ull) : m;
}

__device__ __forceinline__ unsigned long long lane_word(unsigned long long m, int i) {
  return (unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)m, i) |
         (unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(m >> 32), i) << 32;
}

// The walk that suits a set: body(walk kind).
template <typename T, typename F>
__device__ __forceinline__ void with_walk(const EditSet<T>& s, F&& body) {
  if (!s.freq) body(std::integral_constant<int, 0>{});
  else if (s.ncols >= 32) body(std::integral_constant<int, 1>{});
  else body(std::integral_constant<int, 2>{});
}

// Pass 1 of CompactEdits: the flag words, and the non-zero coordinates per block.
template <typename T>
__global__ void __launch_bounds__(64 * kEditWaves) edit_count_kernel(EditJob<T> a, EditJob<T> b) {
  __shared__ unsigned long long red[kEditWaves];
  const EditJob<T> j = (int64_t)blockIdx.x < a.nb ? a : b;
  const int64_t blk = (int64_t)blockIdx.x < a.nb ? blockIdx.x : blockIdx.x - a.nb;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t w0 = blk * kEditChunks + w * kEditWords;
  const int64_t left = j.s.ncoord - w0 * 64;  // coordinates from the wave's first on
  int cnt = 0;
  unsigned long long mine = 0;
  auto word = [&](int i, T v, bool in) {
    const unsigned long long m = __ballot(in && v != T(0));
    cnt += __popcll(m);
    if (lane == i) mine = m;
  };
  with_walk(j.s, [&](auto kind) {
    if (left <= 0) return;
    CoordWalk<T, decltype(kind)::value> at(j.s, w0 * 64, lane);
    if (left >= 64 * kEditWords) {
#pragma unroll
      for (int i0 = 0; i0 < kEditWords; i0 += kEditBatch) {
        T v[kEditBatch];
#pragma unroll
        for (int u = 0; u < kEditBatch; ++u, at.next(lane)) v[u] = *at.ptr();
#pragma unroll
        for (int u = 0; u < kEditBatch; ++u) word(i0 + u, v[u], true);
      }
    } else {
      for (int i = 0; i < kEditWords; ++i, at.next(lane)) {
        const bool in = i * 64 + lane < left;
        word(i, in ? *at.ptr() : T(0), in);
      }
    }
  });
  const int64_t nbytes = (j.s.ncoord + 7) >> 3, b0 = (w0 + lane) * 8;
  if (lane < kEditWords && b0 < nbytes) {
    if (b0 + 8 <= nbytes) *reinterpret_cast<unsigned long long*>(j.flags + b0) = mine;
    else
      for (int k = 0; b0 + k < nbytes; ++k) j.flags[b0 + k] = (uint8_t)(mine >> (8 * k));
  }
  if (lane == 0) red[w] = (unsigned long long)cnt;
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long t = 0;
    for (int i = 0; i < kEditWaves; ++i) t += red[i];
    j.off[blk] = t;
  }
}

// Exclusive scan of n block counts in place (one block of 1024 lanes per set, each lane a
// contiguous run, held in registers where it is short); the total goes to *total.  The block of
// the first set clears the status word when one is given.
struct ScanJob {
  unsigned long long* part;
  int64_t n;
  unsigned long long* total;
};
__global__ void __launch_bounds__(1024) edit_scan_kernel(ScanJob a, ScanJob b, unsigned* status) {
  __shared__ unsigned long long red[16];
  constexpr int R = 8;
  const ScanJob j = blockIdx.x == 0 ? a : b;
  const int t = threadIdx.x;
  if (status && blockIdx.x == 0 && t == 0) *status = 0u;
  const int64_t per = (j.n + 1023) / 1024;
  const int64_t lo = (int64_t)t * per < j.n ? (int64_t)t * per : j.n;
  const int64_t hi = lo + per < j.n ? lo + per : j.n;
  const bool held = per <= R;
  unsigned long long v[R], mine = 0;
  if (held) {
#pragma unroll
    for (int i = 0; i < R; ++i) v[i] = lo + i < hi ? j.part[lo + i] : 0ull;
#pragma unroll
    for (int i = 0; i < R; ++i) mine += v[i];
  } else {
    for (int64_t i = lo; i < hi; ++i) mine += j.part[i];
  }
  // inclusive scan over the lanes of the wave, then over the waves
  unsigned long long inc = mine;
  for (int off = 1; off < 64; off <<= 1) {
    const unsigned long long o = __shfl_up(inc, off, 64);
    if ((t & 63) >= off) inc += o;
  }
  if ((t & 63) == 63) red[t >> 6] = inc;
  __syncthreads();
  unsigned long long wbase = 0;
  for (int i = 0; i < (t >> 6); ++i) wbase += red[i];
  unsigned long long run = wbase + inc - mine;
  if (held) {
#pragma unroll
    for (int i = 0; i < R; ++i) {
      if (lo + i < hi) j.part[lo + i] = run;
      run += v[i];
    }
  } else {
    for (int64_t i = lo; i < hi; ++i) {
      const unsigned long long x = j.part[i];
      j.part[i] = run;
      run += x;
    }
  }
  if (t == 1023) *j.total = run;
}

// Status bits the coding kernels raise (OR-ed into one word).
constexpr unsigned kEditCodeRange = 1u;  // a code outside int32 (or a non-zero edit with a zero step)
constexpr unsigned kEditFlagCount = 2u;  // decoder: set flags and given code count disagree

// Position of the first code of each of the wave's words: lane i < kEditWords gets word i's.
__device__ __forceinline__ unsigned long long word_bases(unsigned long long m, unsigned long long first,
                                                         unsigned long long* lds) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int own = __popcll(m);
  int inc = own;
#pragma unroll
  for (int off = 1; off < kEditWords; off <<= 1) {
    const int o = __shfl_up(inc, off, 64);
    if (lane >= off) inc += o;
  }
  if (lane == kEditWords - 1) lds[w] = (unsigned long long)inc;
  __syncthreads();
  for (int i = 0; i < w; ++i) first += lds[i];
  return first + (unsigned long long)(inc - own);
}

// Pass 2 of CompactEdits fused with QuantizeEdits: the codes of the flagged coordinates.
template <typename T>
__global__ void __launch_bounds__(64 * kEditWaves) edit_write_kernel(EditJob<T> a, EditJob<T> b, unsigned* status) {
  __shared__ unsigned long long red[kEditWaves];
  __shared__ T packed[kEditWaves][64 * kEditWords];
  const EditJob<T> j = (int64_t)blockIdx.x < a.nb ? a : b;
  const int64_t blk = (int64_t)blockIdx.x < a.nb ? blockIdx.x : blockIdx.x - a.nb;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t w0 = blk * kEditChunks + w * kEditWords;
  const unsigned long long words = load_words(j.flags, j.s.ncoord, w0, lane);
  const unsigned long long bases = word_bases(words, j.off[blk], red);
  const double step = j.step;
  // the wave's flagged values, packed in LDS first: their division (FP64) and stores then run on
  // full waves, however sparse the flags are
  const unsigned long long first = lane_word(bases, 0);
  const int n = (int)(lane_word(bases, kEditWords - 1) - first) + __popcll(lane_word(words, kEditWords - 1));
  T* const mine = packed[w];
  with_walk(j.s, [&](auto kind) {
    CoordWalk<T, decltype(kind)::value> at(j.s, w0 * 64, lane);
#pragma unroll
    for (int i0 = 0; i0 < kEditWords; i0 += kEditBatch) {
      T v[kEditBatch];
#pragma unroll
      for (int u = 0; u < kEditBatch; ++u, at.next(lane)) {
        v[u] = T(0);
        if ((lane_word(words, i0 + u) >> lane) & 1ull) v[u] = *at.ptr();
      }
#pragma unroll
      for (int u = 0; u < kEditBatch; ++u) {
        const unsigned long long m = lane_word(words, i0 + u);
        if ((m >> lane) & 1ull) mine[(int)(lane_word(bases, i0 + u) - first) + lane_prefix(m)] = v[u];
      }
    }
  });
  __syncthreads();
  unsigned bad = 0;
  int32_t* const codes = j.codes + first;
  for (int i = lane; i < n; i += 64) {
    const double q = step > 0.0 ? rint((double)mine[i] / step) : 0.0;
    if (!(step > 0.0) || !(fabs(q) < 2147483648.0)) bad |= kEditCodeRange;
    codes[i] = (int32_t)(fabs(q) < 2147483648.0 ? q : 0.0);
  }
  if (bad) atomicOr(status, bad);
}

// Decoder pass 1: set flags per block, a wave per block.
template <typename T>
__global__ void __launch_bounds__(256) flag_count_kernel(EditJob<T> a, EditJob<T> b) {
  static_assert(kEditChunks == 64, "a lane per flag word");
  const int lane = threadIdx.x & 63;
  const int64_t g = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (g >= a.nb + b.nb) return;
  const EditJob<T> j = g < a.nb ? a : b;
  const int64_t blk = g < a.nb ? g : g - a.nb;
  unsigned long long cnt = 0;
  for (int k = 0; k < kEditChunks / kEditWords; ++k)
    if (lane / kEditWords == k)
      cnt = (unsigned long long)__popcll(load_words(j.flags, j.s.ncoord, blk * kEditChunks + k * kEditWords, lane % kEditWords));
  cnt = wave_sum_u64(cnt);
  if (lane == 0) j.off[blk] = cnt;
}

// Decoder pass 2: dense dequantised edits, code * step at flagged coordinates and 0
// elsewhere, written as TO at the set's offsets (spatial: the output field; frequency:
// the spectrum buffer).  Codes past ncodes are never read: every position is below the flag
// count, which is checked.
template <typename TO>
__global__ void __launch_bounds__(64 * kEditWaves) edit_expand_kernel(EditJob<TO> a, EditJob<TO> b, unsigned* status) {
  __shared__ unsigned long long red[kEditWaves];
  const EditJob<TO> j = (int64_t)blockIdx.x < a.nb ? a : b;
  const int64_t blk = (int64_t)blockIdx.x < a.nb ? blockIdx.x : blockIdx.x - a.nb;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (*j.total != (unsigned long long)j.ncodes) {
    if (blk == 0 && threadIdx.x == 0) atomicOr(status, kEditFlagCount);
    return;
  }
  const int64_t w0 = blk * kEditChunks + w * kEditWords;
  const unsigned long long words = load_words(j.flags, j.s.ncoord, w0, lane);
  const unsigned long long bases = word_bases(words, j.off[blk], red);
  const int64_t left = j.s.ncoord - w0 * 64;
  if (left <= 0) return;
  auto value = [&](int i) -> int32_t {  // the code of this lane's coordinate of word i, 0 where not set
    const unsigned long long m = lane_word(words, i);
    const int32_t* const codes = j.codes + lane_word(bases, i);
    int32_t q = 0;
    if ((m >> lane) & 1ull) q = codes[(uint32_t)lane_prefix(m)];
    return q;
  };
  with_walk(j.s, [&](auto kind) {
    CoordWalk<TO, decltype(kind)::value> at(j.s, w0 * 64, lane);
#pragma unroll
    for (int i0 = 0; i0 < kEditWords; i0 += kEditBatch) {
      int32_t q[kEditBatch];
#pragma unroll
      for (int u = 0; u < kEditBatch; ++u) q[u] = value(i0 + u);
#pragma unroll
      for (int u = 0; u < kEditBatch; ++u, at.next(lane))
        if ((i0 + u) * 64 + lane < left) *at.ptr() = q[u] ? (TO)((double)q[u] * j.step) : TO(0);
    }
  });
}

// Dense copy of a coordinate set (the accumulators in coordinate order).
template <typename T>
__global__ void __launch_bounds__(256) edit_export_kernel(EditSet<T> s, T* out) {
  const int64_t c = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (c < s.ncoord) out[c] = s.val[edit_offset(s, c)];
}

// Fill n values of T with zero (the frequency accumulators before the loop; a kernel, so
// that a captured stream records no memset node), 16 bytes a lane.
template <typename T>
__global__ void __launch_bounds__(256) zero_fill_kernel(T* p, int64_t n) {
  constexpr int V = 16 / (int)sizeof(T);  // p is 256-byte aligned
  const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * V;
  if (i + V <= n) *reinterpret_cast<float4*>(p + i) = make_float4(0.f, 0.f, 0.f, 0.f);
  else
    for (int k = 0; i + k < n; ++k) p[i + k] = T(0);
}

}  // namespace ffcz
