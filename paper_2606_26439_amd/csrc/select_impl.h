// select_impl.h -- workgroup-wide exact top-k over 64-bit ranking keys.
//
// A ranking key orders entries exactly as the top-k contract requires
// (score descending, then id ascending): the high 32 bits are the score's
// bits made order-preserving as an unsigned integer (NaN -> 0, below -inf),
// the low 32 bits are ~id. Key 0 never belongs to a real entry (ids are below
// 2^31, so ~id >= 2^31) and serves as padding that ranks below everything.
//
// block_topk() finds the k largest keys of n entries, enumerated by callables
// of their high and low words, with a radix select: starting from the bits all keys
// share, 12-bit digits fix a key prefix until the entries above the prefix
// plus the entries on it fit the sort buffer; those are collected and sorted
// by a bitonic network. Integer
// keys only, so the result does not depend on the launch shape or on the
// order in which entries are visited.
#pragma once
#include "device_common.h"

namespace topk_detail {

__device__ __forceinline__ uint32_t score_key(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7FFFFFFFu) > 0x7F800000u) return 0u;  // NaN ranks last
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ __forceinline__ float key_score(uint32_t k) {
  return __uint_as_float((k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k);
}

__device__ __forceinline__ uint64_t rank_key(uint32_t sk, uint32_t id) {
  return ((uint64_t)sk << 32) | (uint64_t)(0xFFFFFFFFu - id);
}

__device__ __forceinline__ int32_t key_id(uint64_t key) {
  return (int32_t)(0xFFFFFFFFu - (uint32_t)key);
}

constexpr int SEL_BINS = 4096;
// LDS words of block_topk's histogram area: the bins and a few result words
// (bin, count above it, two collection counters, then 16 wave totals)
constexpr int SEL_HIST_WORDS = SEL_BINS + 24;

// Inclusive prefix sum over the 64 lanes of a wave.
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v) {
  const int lane = lane_id();
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    uint32_t o = __shfl_up(v, off, 64);
    if (lane >= off) v += o;
  }
  return v;
}

// The bin holding the rem-th largest entry of a SEL_BINS-bin histogram
// (1 <= rem <= total count) and the number of entries in higher bins; every
// thread of the workgroup gets the same answer. hist[SEL_BINS ..] is scratch.
__device__ __forceinline__ void select_bin(uint32_t* hist, uint32_t rem, uint32_t& bin, uint32_t& above) {
  const int t = threadIdx.x, nt = blockDim.x;
  const int per = SEL_BINS / nt;  // nt divides SEL_BINS (256, 512 or 1024)
  const int hi = SEL_BINS - t * per;  // thread t: bins [hi - per, hi), high to low
  uint32_t local = 0;
  for (int b = hi - 1; b >= hi - per; --b) local += hist[b];
  // exclusive prefix over threads in thread order (= bins high to low)
  const uint32_t incl = wave_incl_scan(local);
  const int w = t >> 6;
  uint32_t* wave_tot = hist + SEL_BINS + 8;  // at most 16 waves
  if ((t & 63) == 63) wave_tot[w] = incl;
  __syncthreads();
  uint32_t base = 0;
  for (int i = 0; i < w; ++i) base += wave_tot[i];
  uint32_t run = base + incl - local;
  if (run < rem && run + local >= rem) {
    for (int b = hi - 1; b >= hi - per; --b) {
      const uint32_t h = hist[b];
      if (run + h >= rem) {
        hist[SEL_BINS] = (uint32_t)b;
        hist[SEL_BINS + 1] = run;
        break;
      }
      run += h;
    }
  }
  __syncthreads();
  bin = hist[SEL_BINS];
  above = hist[SEL_BINS + 1];
  __syncthreads();
}

// The value of lane i ^ M of the wave (M a power of two below 64): quad
// permutes for 1 and 2, a half-row mirror with a quad mirror for 4, a row
// rotation for 8 (no LDS round trip), shuffles for 16 and 32.
template <int M>
__device__ __forceinline__ uint32_t lane_xor(uint32_t v) {
  if constexpr (M == 1)
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, false);
  else if constexpr (M == 2)
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, false);
  else if constexpr (M == 4)  // i ^ 7, then i ^ 3
    return (uint32_t)__builtin_amdgcn_update_dpp(
        0, __builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, false), 0x1B, 0xF, 0xF, false);
  else if constexpr (M == 8)
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x128, 0xF, 0xF, false);
  else
    return (uint32_t)__shfl_xor((int)v, M, 64);
}
template <int M>
__device__ __forceinline__ uint64_t lane_xor64(uint64_t v) {
  return ((uint64_t)lane_xor<M>((uint32_t)(v >> 32)) << 32) | lane_xor<M>((uint32_t)v);
}

// One exchange step of a bitonic network between lanes: v becomes the larger
// (where the lower lane of a descending pair holds it) or the smaller of v
// and lane i ^ M's value.
template <int M>
__device__ __forceinline__ void lane_exchange(uint64_t& v, bool desc) {
  const uint64_t o = lane_xor64<M>(v);
  const bool take_max = ((lane_id() & M) == 0) == desc;
  v = (v < o) == take_max ? o : v;
}
// The steps of strides 32 to 1: merges 64 lanes' bitonic sequence.
__device__ __forceinline__ void wave_merge(uint64_t& v, bool desc) {
  lane_exchange<32>(v, desc);
  lane_exchange<16>(v, desc);
  lane_exchange<8>(v, desc);
  lane_exchange<4>(v, desc);
  lane_exchange<2>(v, desc);
  lane_exchange<1>(v, desc);
}

// Bitonic sort, descending, of E keys per thread (key e of thread t is element
// e * nt + t of n = E * nt; with E = 1, n <= nt, a multiple of 64, and the
// threads past n only join the barriers). Exchanges stay in registers where
// partners share a thread or a wave, with constant strides, and go through
// LDS only between waves: 1024 keys on 1024 threads take 10 LDS exchanges
// instead of 55 passes with a barrier each.
template <int E>
__device__ __forceinline__ void bitonic_regs(uint64_t* keys, int n) {
  const int t = threadIdx.x, nt = blockDim.x;
  const bool live = t < n;
  uint64_t v[E];
#pragma unroll
  for (int e = 0; e < E; ++e) v[e] = live ? keys[e * nt + t] : 0ull;
#pragma unroll
  for (int e = 0; e < E; ++e) {  // blocks of 2 to 64 (e * nt does not touch their bits)
    lane_exchange<1>(v[e], (t & 2) == 0);
    lane_exchange<2>(v[e], (t & 4) == 0);
    lane_exchange<1>(v[e], (t & 4) == 0);
    lane_exchange<4>(v[e], (t & 8) == 0);
    lane_exchange<2>(v[e], (t & 8) == 0);
    lane_exchange<1>(v[e], (t & 8) == 0);
    lane_exchange<8>(v[e], (t & 16) == 0);
    lane_exchange<4>(v[e], (t & 16) == 0);
    lane_exchange<2>(v[e], (t & 16) == 0);
    lane_exchange<1>(v[e], (t & 16) == 0);
    lane_exchange<16>(v[e], (t & 32) == 0);
    lane_exchange<8>(v[e], (t & 32) == 0);
    lane_exchange<4>(v[e], (t & 32) == 0);
    lane_exchange<2>(v[e], (t & 32) == 0);
    lane_exchange<1>(v[e], (t & 32) == 0);
    wave_merge(v[e], (t & 64) == 0);
  }
  for (int size = 128; size <= n; size <<= 1) {
    for (int stride = size >> 1; stride >= 64; stride >>= 1) {
      uint64_t o[E];
      if (E == 1 || stride < nt) {
        __syncthreads();  // earlier reads of the exchange area are done
        if (live) {
#pragma unroll
          for (int e = 0; e < E; ++e) keys[e * nt + t] = v[e];
        }
        __syncthreads();
#pragma unroll
        for (int e = 0; e < E; ++e) o[e] = live ? keys[(e * nt + t) ^ stride] : 0ull;
      } else {
        const int f = stride / nt;  // partners in this thread
#pragma unroll
        for (int e = 0; e < E; ++e) {
          o[e] = v[e];
#pragma unroll
          for (int q = 1; q < E; q <<= 1)
            if (f == q) o[e] = v[e ^ q];
        }
      }
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const int i = e * nt + t;
        const bool take_max = ((i & stride) == 0) == ((i & size) == 0);
        v[e] = (v[e] < o[e]) == take_max ? o[e] : v[e];
      }
    }
#pragma unroll
    for (int e = 0; e < E; ++e) wave_merge(v[e], ((e * nt + t) & size) == 0);
  }
  __syncthreads();
  if (live) {
#pragma unroll
    for (int e = 0; e < E; ++e) keys[e * nt + t] = v[e];
  }
  __syncthreads();
}

// Sorts n (a power of two, n >= 64) keys descending in LDS, whole workgroup,
// the keys being visible to it: in registers up to MAXE keys per thread, else
// by passes over LDS (MAXE is small where many kernels carry the code).
template <int MAXE>
__device__ __forceinline__ void bitonic_desc(uint64_t* keys, int n) {
  const int nt = blockDim.x;
  if (n <= nt) return bitonic_regs<1>(keys, n);
  if constexpr (MAXE >= 2)
    if (n == 2 * nt) return bitonic_regs<2>(keys, n);
  if constexpr (MAXE >= 4)
    if (n == 4 * nt) return bitonic_regs<4>(keys, n);
  for (int size = 2; size <= n; size <<= 1) {
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      for (int i = threadIdx.x; i < n; i += nt) {
        const int j = i ^ stride;
        if (j > i) {
          const bool desc = (i & size) == 0;
          const uint64_t x = keys[i], y = keys[j];
          if (desc ? (x < y) : (x > y)) {
            keys[i] = y;
            keys[j] = x;
          }
        }
      }
      __syncthreads();
    }
  }
}

// The min(k, n) largest of the keys (hi(i) << 32 | lo(i)), i in [0, n), sorted
// descending, into out[0 ..); returns that count. Whole workgroup; hist has
// SEL_HIST_WORDS words and buf `cap` keys of LDS (cap a power of two,
// cap >= k, cap >= 64). lo (an id, often from memory) is
// read only for keys that a pass over the score bits leaves in question.
template <int MAXE, class Hi, class Lo>
__device__ __forceinline__ int block_topk(int64_t n, int k, Hi hi, Lo lo, uint32_t* hist, uint64_t* buf, int cap,
                          uint64_t* out) {
  auto get = [&](int64_t i) -> uint64_t { return ((uint64_t)hi(i) << 32) | lo(i); };
  const int t = threadIdx.x, nt = blockDim.x;
  int count;
  if (n <= cap) {
    int p2 = 64;
    while (p2 < n) p2 <<= 1;
    for (int i = t; i < p2; i += nt) buf[i] = i < n ? get((int64_t)i) : 0ull;
    __syncthreads();
    bitonic_desc<MAXE>(buf, p2);
    count = n < k ? (int)n : k;
  } else {
    // The score bits every key shares (where the largest and the smallest
    // score key agree) start the prefix, so the first digit already splits
    // the keys: without this, keys of scores in a narrow range all fall into
    // one or two bins of the top digit and their histogram atomics serialise.
    uint32_t hmax = 0u, hmin = ~0u;
    for (int64_t i = t; i < n; i += nt) {
      const uint32_t h = hi(i);
      hmax = h > hmax ? h : hmax;
      hmin = h < hmin ? h : hmin;
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) {
      const uint32_t a = (uint32_t)__shfl_xor((int)hmax, m, 64);
      const uint32_t b = (uint32_t)__shfl_xor((int)hmin, m, 64);
      hmax = a > hmax ? a : hmax;
      hmin = b < hmin ? b : hmin;
    }
    // wave partials in the first 32 words of hist, before the bins are used
    const int w = t >> 6, nw = nt >> 6;
    if ((t & 63) == 0) {
      hist[w] = hmax;
      hist[16 + w] = hmin;
    }
    __syncthreads();
    for (int i = 0; i < nw; ++i) {
      hmax = hist[i] > hmax ? hist[i] : hmax;
      hmin = hist[16 + i] < hmin ? hist[16 + i] : hmin;
    }
    __syncthreads();
    int plen = hmax == hmin ? 32 : __builtin_clz(hmax ^ hmin);  // key bits fixed by the prefix
    const uint64_t kmax = (uint64_t)hmax << 32;
    uint64_t prefix = plen == 0 ? 0ull : kmax >> (64 - plen);
    uint32_t rem = (uint32_t)k, n_above = 0;
    while (plen < 64) {
      // digits end at the boundary of the score bits
      const int left = plen < 32 ? 32 - plen : 64 - plen;
      const int dbits = left < 12 ? left : 12;
      const int shift = 64 - plen - dbits;
      const uint64_t dmask = (1ull << dbits) - 1ull;
      // keys on the prefix: (key & pmask) == pbits (no shift by 64)
      const uint64_t pmask = plen == 0 ? 0ull : ~0ull << (64 - plen);
      const uint64_t pbits = plen == 0 ? 0ull : prefix << (64 - plen);
      for (int i = t; i < SEL_BINS; i += nt) hist[i] = 0u;
      __syncthreads();
      if (plen < 32) {
        for (int64_t i = t; i < n; i += nt) {
          const uint64_t key = (uint64_t)hi(i) << 32;
          if ((key & pmask) == pbits) atomicAdd(&hist[(key >> shift) & dmask], 1u);
        }
      } else {
        const uint32_t on = (uint32_t)(pbits >> 32);
        for (int64_t i = t; i < n; i += nt) {
          if (hi(i) != on) continue;
          const uint64_t key = get(i);
          if ((key & pmask) == pbits) atomicAdd(&hist[(key >> shift) & dmask], 1u);
        }
      }
      __syncthreads();
      uint32_t bin, above;
      select_bin(hist, rem, bin, above);
      const uint32_t on_bin = hist[bin];
      __syncthreads();
      n_above += above;
      rem -= above;
      prefix = (prefix << dbits) | bin;
      plen += dbits;
      if (n_above + on_bin <= (uint32_t)cap) break;
    }
    // entries above the prefix (n_above < k of them) go to the front, the
    // entries on it after them, as many as fit (past the last digit they are
    // equal keys, so which of them are kept does not matter)
    if (t == 0) {
      hist[SEL_BINS + 2] = 0u;
      hist[SEL_BINS + 3] = 0u;
    }
    __syncthreads();
    // the prefix and each key's top plen bits, aligned at the top
    const uint64_t tmask = plen == 64 ? ~0ull : ~(~0ull >> plen);
    const uint64_t pbits = plen == 64 ? prefix : prefix << (64 - plen);
    const uint32_t least = (uint32_t)(pbits >> 32);
    for (int64_t i = t; i < n; i += nt) {
      if (hi(i) < least) continue;  // below the prefix
      const uint64_t key = get(i);
      const uint64_t top = key & tmask;
      if (top > pbits) {
        buf[atomicAdd(&hist[SEL_BINS + 2], 1u)] = key;
      } else if (top == pbits) {
        const uint32_t s = atomicAdd(&hist[SEL_BINS + 3], 1u);
        if (n_above + s < (uint32_t)cap) buf[n_above + s] = key;
      }
    }
    __syncthreads();
    const uint32_t on = hist[SEL_BINS + 3];
    const int got = (int)(n_above + on < (uint32_t)cap ? n_above + on : (uint32_t)cap);
    int p2 = 64;
    while (p2 < got) p2 <<= 1;
    for (int i = got + t; i < p2; i += nt) buf[i] = 0ull;
    __syncthreads();
    bitonic_desc<MAXE>(buf, p2);
    count = k;
  }
  for (int i = t; i < count; i += nt) out[i] = buf[i];
  __syncthreads();
  return count;
}

}  // namespace topk_detail
