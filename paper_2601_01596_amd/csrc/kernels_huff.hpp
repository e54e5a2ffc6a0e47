// Lossless coding of the edit streams (Alg. 1, LosslesslyCompressEdits; Sec. IV-B, IV-D):
// symbols (flag bytes or int32 codes) are counted blockwise into a global frequency table,
// the host builds the Huffman code from that table, and the stream is encoded in parallel:
// every symbol's bit offset is an exclusive prefix sum of code lengths (block sums, one-block
// scan, block-local scan), and a block puts its codes together in LDS and stores whole words.
//
// Stream layout (bits): codes most significant bit first, each 32-bit word filled from its
// top bit down.  The offset of every kHuffChunk-th symbol is kept, so the decoder runs one
// lane per chunk of symbols, each from its own starting bit.
#pragma once
#include <climits>

#include "common.hpp"

namespace ffcz {

constexpr int kHuffChunk = 256;       // symbols per decoder chunk
constexpr int kHuffBlock = 256;       // lanes per block
constexpr int kHuffPerLane = 16;      // consecutive symbols per lane: one 16-byte load of flag bytes
constexpr int64_t kHuffBlockSyms = (int64_t)kHuffBlock * kHuffPerLane;
constexpr int kHuffLdsBins = 8192;    // alphabets up to this size count in LDS
constexpr int kHuffLdsTab = 2048;     // alphabets up to this size keep their code table in LDS
constexpr int kHuffDecBlock = 64;     // decoder lanes per block (one chunk each): small blocks
                                      // spread the few chunks of a stream over more CUs
constexpr int kHuffHistBlock = 1024;  // lanes of a counting block

// Bins (symbol - lo) of the 16 symbols from i0 on, -1 past the end.  W: 1-byte or 4-byte signed
// symbols; vec: the stream starts on a 16-byte boundary, so whole groups are 16-byte loads.
template <int W>
__device__ __forceinline__ void huff_load(const void* s, int64_t i0, int64_t n, int64_t lo, int vec, int (&v)[16]) {
  if (vec && i0 + 16 <= n) {
    if constexpr (W == 1) {
      const uint4 q = *reinterpret_cast<const uint4*>((const uint8_t*)s + i0);
      const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
      for (int k = 0; k < 16; ++k) v[k] = (int)((w[k >> 2] >> (8 * (k & 3))) & 255u) - (int)lo;
    } else {
      const int4* p = reinterpret_cast<const int4*>((const int32_t*)s + i0);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int4 q = p[k];
        v[4 * k] = (int)(q.x - lo);
        v[4 * k + 1] = (int)(q.y - lo);
        v[4 * k + 2] = (int)(q.z - lo);
        v[4 * k + 3] = (int)(q.w - lo);
      }
    }
    return;
  }
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    v[k] = -1;
    if (i0 + k < n)
      v[k] = (int)((W == 1 ? (int64_t)((const uint8_t*)s)[i0 + k] : (int64_t)((const int32_t*)s)[i0 + k]) - lo);
  }
}

// Block minima and maxima of the symbols.  Bound by the read (16 M flag bytes: 27 us with a load
// per byte, 6 us with 16-byte loads).
template <int W>
__global__ void __launch_bounds__(kHuffBlock) huff_minmax_kernel(const void* s, int64_t n, int vec, long long* part) {
  __shared__ long long rmin[4], rmax[4];
  long long mn = LLONG_MAX, mx = LLONG_MIN;
  auto take = [&](long long x) {
    mn = x < mn ? x : mn;
    mx = x > mx ? x : mx;
  };
  for (int64_t g = (int64_t)blockIdx.x * kHuffBlock + threadIdx.x; 16 * g < n; g += (int64_t)gridDim.x * kHuffBlock) {
    const int64_t i0 = 16 * g;
    if (vec && i0 + 16 <= n) {
      int a = INT_MAX, b = INT_MIN;
      if constexpr (W == 1) {
        int v[16];
        huff_load<1>(s, i0, n, 0, vec, v);
#pragma unroll
        for (int k = 0; k < 16; ++k) {
          a = v[k] < a ? v[k] : a;
          b = v[k] > b ? v[k] : b;
        }
      } else {
        const int4* p = reinterpret_cast<const int4*>((const int32_t*)s + i0);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int4 q = p[k];
          a = min(min(a, min(q.x, q.y)), min(q.z, q.w));
          b = max(max(b, max(q.x, q.y)), max(q.z, q.w));
        }
      }
      take(a);
      take(b);
    } else {
      for (int64_t i = i0; i < n && i < i0 + 16; ++i)
        take(W == 1 ? (long long)((const uint8_t*)s)[i] : (long long)((const int32_t*)s)[i]);
    }
  }
  for (int off = 32; off > 0; off >>= 1) {
    const long long a = __shfl_xor(mn, off, 64), b = __shfl_xor(mx, off, 64);
    mn = a < mn ? a : mn;
    mx = b > mx ? b : mx;
  }
  if ((threadIdx.x & 63) == 0) {
    rmin[threadIdx.x >> 6] = mn;
    rmax[threadIdx.x >> 6] = mx;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 4; ++w) {
      mn = rmin[w] < mn ? rmin[w] : mn;
      mx = rmax[w] > mx ? rmax[w] : mx;
    }
    part[2 * blockIdx.x] = mn;
    part[2 * blockIdx.x + 1] = mx;
  }
}

// The global frequency table over lo .. lo + nalpha - 1 (counts must start at zero): small
// alphabets count per block in LDS and add the block's table once, larger ones add straight
// into the global table.  Integer additions, so the table does not depend on the order.  Edit
// streams are dominated by one symbol (zero flag bytes, zero codes), whose atomics would
// serialise, so each wave counts one symbol by ballots, chosen anew for every 1024 symbols: the
// commonest of a sample of 64 (from different places of the lanes' groups), of up to four tried.
// Every block adds its whole table at the end (about 6 G additions/s over all blocks), so there are
// few and large ones.  16 M flags with 2 % of the bits set 15 us, with 20 % 19 us, 1 M codes over
// 8000 symbols 8 us.  (The symbol that the block meets first counted in registers instead: 51, 21 and
// 8 us, the blocks that began with a rarer symbol being waited for; 64 M codes with the rare symbol at
// every block's head 226 us, now 41.)
constexpr int kHuffVotes = 4;
template <int W>
__global__ void __launch_bounds__(kHuffHistBlock) huff_hist_kernel(const void* s, int64_t n, int64_t lo,
                                                                   int64_t nalpha, int vec,
                                                                   unsigned long long* counts) {
  extern __shared__ unsigned int h[];  // nalpha bins where they fit
  const bool local = nalpha <= kHuffLdsBins;
  const int lane = threadIdx.x & 63;
  if (local)
    for (int i = threadIdx.x; i < nalpha; i += kHuffHistBlock) h[i] = 0u;
  __syncthreads();
  constexpr int64_t step = (int64_t)kHuffHistBlock * kHuffPerLane;
  for (int64_t b = (int64_t)blockIdx.x * step; b < n; b += (int64_t)gridDim.x * step) {
    int v[16];
    huff_load<W>(s, b + (int64_t)threadIdx.x * kHuffPerLane, n, lo, vec, v);
    int pick = v[0];
#pragma unroll
    for (int k = 1; k < 16; ++k) pick = (lane & 15) == k ? v[k] : pick;
    int dom = -1, best = 0;
    unsigned long long left = __ballot(pick >= 0);
    for (int t = 0; t < kHuffVotes && __popcll(left) > best; ++t) {
      const int c = __builtin_amdgcn_readlane(pick, __ffsll((long long)left) - 1);
      const unsigned long long m = __ballot(pick == c);
      if (__popcll(m) > best) {
        best = __popcll(m);
        dom = c;
      }
      left &= ~m;
    }
    unsigned int nd = 0;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      const bool is = v[k] == dom;
      nd += (unsigned int)__popcll(__ballot(is));
      if (!is && v[k] >= 0) {
        if (local) atomicAdd(&h[v[k]], 1u);
        else atomicAdd(&counts[v[k]], 1ull);
      }
    }
    if (lane == 0 && dom >= 0) {
      if (local) atomicAdd(&h[dom], nd);
      else atomicAdd(&counts[dom], (unsigned long long)nd);
    }
  }
  if (local) {
    __syncthreads();
    for (int i = threadIdx.x; i < nalpha; i += kHuffHistBlock)
      if (h[i]) atomicAdd(&counts[i], (unsigned long long)h[i]);
  }
}

// Bits of the symbols of each block of kHuffBlockSyms symbols.
template <int W>
__global__ void __launch_bounds__(kHuffBlock) huff_bits_kernel(const void* s, int64_t n, int64_t lo, int64_t nalpha,
                                                               int vec, const uint8_t* len, unsigned long long* part) {
  __shared__ unsigned int red[4];
  __shared__ uint8_t tl[kHuffLdsTab];
  const bool lt = nalpha <= kHuffLdsTab;
  if (lt) {
    for (int i = threadIdx.x; i < nalpha; i += kHuffBlock) tl[i] = len[i];
    __syncthreads();
  }
  int v[16];
  huff_load<W>(s, (int64_t)blockIdx.x * kHuffBlockSyms + (int64_t)threadIdx.x * kHuffPerLane, n, lo, vec, v);
  unsigned int b = 0;
#pragma unroll
  for (int k = 0; k < 16; ++k)
    if (v[k] >= 0) b += lt ? tl[v[k]] : len[v[k]];
  for (int off = 32; off > 0; off >>= 1) b += __shfl_xor(b, off, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = b;
  __syncthreads();
  if (threadIdx.x == 0) part[blockIdx.x] = (unsigned long long)red[0] + red[1] + red[2] + red[3];
}

// Encode: lane t of a block owns 16 consecutive symbols, so its bit offset is the block offset
// plus an exclusive scan of the lanes' bit counts.  The lane packs its codes into 32-bit words in
// registers and ORs each into the block's words in LDS; the block stores its words, the first
// and last of which it may share with its neighbours, with a global OR (words start at zero).
// The lane holding symbol j * kHuffChunk records that symbol's offset.  Bound by the symbols'
// table look-ups now (16 M flags: 375 us with one or two global ORs per symbol, 20 us).
template <int W>
__global__ void __launch_bounds__(kHuffBlock) huff_encode_kernel(const void* s, int64_t n, int64_t lo, int64_t nalpha,
                                                                 int vec, const uint8_t* len, const uint32_t* code,
                                                                 const unsigned long long* boff, unsigned int* words,
                                                                 unsigned long long* chunk_bits) {
  __shared__ unsigned int wsum[4];
  __shared__ unsigned int ow[kHuffBlockSyms + 1];  // at most 32 bits a symbol
  __shared__ uint32_t tc[kHuffLdsTab];
  __shared__ uint8_t tl[kHuffLdsTab];
  const bool lt = nalpha <= kHuffLdsTab;
  const int t = threadIdx.x;
  if (lt) {
    for (int i = t; i < nalpha; i += kHuffBlock) {
      tc[i] = code[i];
      tl[i] = len[i];
    }
    __syncthreads();
  }
  const int64_t i0 = (int64_t)blockIdx.x * kHuffBlockSyms + (int64_t)t * kHuffPerLane;
  int v[16];
  huff_load<W>(s, i0, n, lo, vec, v);
  int l[16];
  unsigned int mine = 0;
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    l[k] = v[k] >= 0 ? (int)(lt ? tl[v[k]] : len[v[k]]) : 0;
    mine += l[k];
  }
  // inclusive scan over the wave, then over the four waves
  unsigned int inc = mine;
  for (int off = 1; off < 64; off <<= 1) {
    const unsigned int o = __shfl_up(inc, off, 64);
    if ((t & 63) >= off) inc += o;
  }
  if ((t & 63) == 63) wsum[t >> 6] = inc;
  __syncthreads();
  unsigned int rel = inc - mine, total = 0;
  for (int w = 0; w < 4; ++w) {
    rel += w < (t >> 6) ? wsum[w] : 0u;
    total += wsum[w];
  }
  const unsigned long long start = boff[blockIdx.x];  // the block's first bit
  const int sh0 = (int)(start & 31);
  const int nw = (int)((sh0 + total + 31) >> 5);
  for (int i = t; i < nw; i += kHuffBlock) ow[i] = 0u;
  __syncthreads();
  if (i0 < n && i0 % kHuffChunk == 0) chunk_bits[i0 / kHuffChunk] = start + rel;
  unsigned int p = (unsigned int)sh0 + rel;
  int wi = (int)(p >> 5), fill = (int)(p & 31);
  unsigned long long acc = 0;  // top half: the bits of word wi so far
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    if (l[k] == 0) continue;
    const unsigned long long c = lt ? tc[v[k]] : code[v[k]];
    acc |= (c << (64 - l[k])) >> fill;
    fill += l[k];
    if (fill >= 32) {
      atomicOr(&ow[wi], (unsigned int)(acc >> 32));
      acc <<= 32;
      fill -= 32;
      ++wi;
    }
  }
  if ((unsigned int)(acc >> 32)) atomicOr(&ow[wi], (unsigned int)(acc >> 32));
  __syncthreads();
  unsigned int* out = words + (start >> 5);
  for (int i = t; i < nw; i += kHuffBlock) {
    if (i == 0 || i == nw - 1) atomicOr(&out[i], ow[i]);
    else out[i] = ow[i];
  }
}

// Decode: one lane per chunk walks its symbols from the chunk's first bit.  With v the next 32 bits
// of the stream, the code length is the smallest l with v <= top[l], the left-justified last
// code of length l followed by ones (a length without codes repeats the one before; the last
// entry of a full code is 2^32 - 1), and the symbol is sorted[off[l] + (v >> (32 - l))], symbols
// ordered by length, then value.  A lane's chain is read, compare, advance, 256 times, and a
// stream holds few waves (one per 16 K symbols), so what counts is that chain's length and that
// no lane makes the others wait: the limits of all NL lengths from lmin on are compared in turn
// without a branch (they are kernel arguments), the chunks of a block lie side by side in the
// stream, so the block copies its stretch to LDS (up to stage words; a wave whose chunks reach
// past them reads memory), and the symbols sit in LDS where they fit (nlds > 0).  Symbols leave
// in groups of 16 bytes where vec says that the output starts on such a boundary.  (16 M flags /
// 1 M codes: 163 / 211 us with a limit loop, a global look-up and a store per symbol, 87 / 110 us;
// a 4096-entry look-up table before the limit loop 78 / 189 us.)
struct HuffDec {
  const unsigned int* words;
  int64_t nwords;
  const unsigned long long* chunk_bits;
  unsigned long long nbits;
  int64_t n, lo, nchunks;
  const int32_t* sorted;
  int32_t lmin, nlen, nsorted, stage, nlds, vec;
  void* out;
  unsigned int* bad;
  uint32_t top[32];  // of length lmin + j; past the longest code 2^32 - 1
  uint32_t off[33];  // of length lmin + j (modulo 2^32); 0 past the longest code
};

template <int W, int NL>
__global__ void __launch_bounds__(kHuffDecBlock) huff_decode_kernel(HuffDec d) {
  __shared__ uint32_t off[33];
  extern __shared__ unsigned int st[];  // stage words of the stream, then the symbols as 16 bits
  uint16_t* const so = reinterpret_cast<uint16_t*>(st + d.stage);
  const int t = threadIdx.x;
  if (t < 33) off[t] = d.off[t];
  for (int i = t; i < d.nlds; i += kHuffDecBlock) so[i] = (uint16_t)d.sorted[i];
  const int64_t ch0 = (int64_t)blockIdx.x * kHuffDecBlock;
  const unsigned long long w0 = d.chunk_bits[ch0] >> 5;  // the stretch's first word
  for (int i = t; i < d.stage; i += kHuffDecBlock)
    st[i] = w0 + i < (unsigned long long)d.nwords ? d.words[w0 + i] : 0u;
  __syncthreads();
  const int64_t ch = ch0 + t;
  const int64_t i0 = ch * kHuffChunk;
  if (i0 >= d.n) return;
  const int64_t i1 = i0 + kHuffChunk < d.n ? i0 + kHuffChunk : d.n;
  const unsigned long long p0 = d.chunk_bits[ch], p1 = ch + 1 < d.nchunks ? d.chunk_bits[ch + 1] : d.nbits;
  // in the stretch (offsets out of order, as in a damaged stream, count as outside)
  const bool in = p0 >= (w0 << 5) && p1 >= p0 && (p1 >> 5) + 1 < w0 + (unsigned long long)d.stage;
  // One symbol from the 64 stream bits at word pos >> 5; advances pos.  Nothing here branches on
  // the data: a pattern that is no code takes some symbol and shows in worst (the length's number
  // it matched), so that the next symbol's read does not wait for this one's.
  int worst = 0;
  const uint32_t top_at = (uint32_t)d.nsorted - 1u;
  auto take = [&](unsigned int hi, unsigned int lo_, unsigned int& pos) -> uint32_t {
    const unsigned long long pair = ((unsigned long long)hi << 32) | lo_;
    const unsigned int v = (unsigned int)((pair << (pos & 31)) >> 32);
    int j = 0;
#pragma unroll
    for (int k = 0; k < NL - 1; ++k) j += v > d.top[k] ? 1 : 0;
    const int l = min(d.lmin + j, 32);
    pos += (unsigned)l;
    worst = max(worst, j);
    const uint32_t at = min(off[j] + (v >> (32 - l)), top_at);
    return d.nlds > 0 ? (uint32_t)so[at] : (uint32_t)d.sorted[at];
  };
  const uint32_t lo32 = (uint32_t)d.lo;  // symbols are at most 32 bits wide
  auto emit = [&](auto next) {
    int64_t i = i0;
    if (d.vec) {
      constexpr int G = 16 / W;  // symbols per 16 bytes
      for (; i + G <= i1; i += G) {
        uint32_t q[4] = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int k = 0; k < G; ++k) {
          const uint32_t x = next() + lo32;
          if constexpr (W == 1) q[k >> 2] |= (x & 255u) << (8 * (k & 3));
          else q[k] = x;
        }
        *reinterpret_cast<uint4*>((uint8_t*)d.out + i * W) = make_uint4(q[0], q[1], q[2], q[3]);
      }
    }
    for (; i < i1; ++i) {
      const uint32_t x = next() + lo32;
      if constexpr (W == 1) ((uint8_t*)d.out)[i] = (uint8_t)x;
      else ((int32_t*)d.out)[i] = (int32_t)x;
    }
  };
  if (__all(in)) {
    unsigned int pos = (unsigned int)(p0 - (w0 << 5));
    const unsigned int last = (unsigned int)d.stage - 2;
    emit([&]() -> uint32_t {
      const unsigned int k = min(pos >> 5, last);  // a damaged chunk may run past its end
      return take(st[k], st[k + 1], pos);
    });
  } else {
    unsigned long long w = p0 >> 5;
    unsigned int pos = (unsigned int)(p0 & 31);  // kept below 32 from word w on
    auto word = [&](unsigned long long k) -> unsigned int {
      return k < (unsigned long long)d.nwords ? d.words[k] : 0u;
    };
    emit([&]() -> uint32_t {
      w += pos >> 5;
      pos &= 31u;
      return take(word(w), word(w + 1), pos);
    });
  }
  if (worst >= d.nlen) atomicOr(d.bad, 1u);
}

}  // namespace ffcz
