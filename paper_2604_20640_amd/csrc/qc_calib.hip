// MAD flagging and delay/phase application for gfx950.
//
// MAD (arXiv 2604.20640 Sec. 7, eq. 2): T = median(A) + sigma*1.4826*MAD(A)
// on the visibility amplitude A; flag A > T.  Medians are exact order
// statistics found by radix selection (most significant digit first) over
// the bit patterns of non-negative floats, whose unsigned order equals their
// numeric order: float32 amplitudes and float64 deviations |A - median|.
// The key range comes for free (amplitudes: a min/max taken while they are
// loaded; deviations: [0, the larger deviation of the extreme amplitudes]),
// so bits shared by the whole range need no pass.  Once the digit holding
// the wanted rank contains at most SEL_CAND keys, one pass gathers them and
// one wave ranks them.  Even counts average the two middle order
// statistics; the upper one is read off the same candidates when it lies
// among them (else one counting pass finds it).  Once the digit holding the
// wanted rank has few enough keys for the LDS left over, their values are
// compacted into LDS and the remaining passes scan only them.  One workgroup handles one
// population (1024 threads and 11-bit digits for large populations, one
// wave and 8-bit digits for small ones); large populations get their
// amplitudes formed once by a whole-GPU pass and cached in LDS when they
// fit.  Larger ones still are bounded by a sample and read once (below).
//
// Delay/phase application (Sec. 4.1 step 2 and eq. 1; Sec. 7 delay and phase
// corrections): V_ij[k] *= exp(+i [2 pi f_k (tau_i - tau_j) + phi_i - phi_j]).
// The rotation is formed in float64: cycles = f_k (tau_i - tau_j) +
// (phi_i - phi_j)/(2 pi), reduced modulo 1, then sincospi.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "qc_kernels.h"

namespace qc {

namespace {

// Every float64 step of the threshold is a separately rounded IEEE operation
// (no contraction into fused multiply-adds), so the decisions match a plain
// float64 evaluation of the same expressions bit for bit.
#pragma clang fp contract(off)

struct Pop {
  int64_t base, count, inner_n, s_inner, s_outer;
  __device__ __forceinline__ int64_t off(int64_t i) const {
    // 32-bit division when the index and the inner extent fit (every
    // population but the very largest): a fraction of the 64-bit sequence
    if (i <= 0x7fffffffLL && inner_n <= 0x7fffffffLL) {
      const uint32_t q = (uint32_t)i / (uint32_t)inner_n;
      const uint32_t r = (uint32_t)i - q * (uint32_t)inner_n;
      return base + (int64_t)q * s_outer + (int64_t)r * s_inner;
    }
    return base + (i / inner_n) * s_outer + (i % inner_n) * s_inner;
  }
};

__device__ __forceinline__ float amp_f32(float2 v) {
  const double re = (double)v.x, im = (double)v.y;
  return (float)sqrt(re * re + im * im);
}

// Amplitudes of a population: from an LDS cache when it fits, else from a
// materialised amplitude array, else recomputed from vis.
struct AmpSrc {
  const float2* vis;
  Pop pop;
  const float* cache;  // LDS copy, or the population's slice of the materialised array; may be null
  __device__ __forceinline__ float operator()(int64_t i) const {
    return cache ? cache[i] : amp_f32(vis[pop.off(i)]);
  }
};

// A block-uniform 64-bit value read back from LDS, made wave-uniform for
// the compiler (branches on it hold barriers).
__device__ __forceinline__ int64_t rfl64(int64_t v) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)((uint64_t)v >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

// Block-wide search of the digit that holds rank kk in hist[0..NBINS):
// returns (digit, rank within the digit) through sh[].
template <int NT, int NBINS>
__device__ __forceinline__ void find_digit(const unsigned* hist, int64_t kk, unsigned* wsum,
                                           unsigned long long* sh) {
  constexpr int PER = NBINS / NT;  // bins per thread (>= 1)
  constexpr int NW = NT / 64;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  unsigned loc = 0;
#pragma unroll
  for (int i = 0; i < PER; ++i) loc += hist[t * PER + i];
  unsigned v = loc;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const unsigned n = __shfl_up(v, d);
    if (lane >= d) v += n;
  }
  // each thread adds the totals of the waves before its own (independent
  // broadcast reads instead of one thread's serial prefix and a barrier)
  unsigned before = 0u;
  if (NW > 1) {
    if (lane == 63) wsum[wave] = v;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < NW; ++w) before += w < wave ? wsum[w] : 0u;
  }
  const int64_t incl = (int64_t)v + before;
  const int64_t excl = incl - loc;
  if (excl <= kk && kk < incl) {
    int64_t c = excl;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const unsigned h = hist[t * PER + i];
      if (kk < c + (int64_t)h) {
        sh[0] = (unsigned long long)(t * PER + i);
        sh[1] = (unsigned long long)(kk - c);
        break;
      }
      c += h;
    }
  }
  __syncthreads();
}

// Keys of a selection that are still candidates once few remain: they are
// gathered and ranked by one wave instead of further histogram passes.
constexpr int SEL_CAND = 64;

// fn(i, key(i)) for this thread's elements i = threadIdx.x + NT j.  The
// large-population kernel forms its keys in batches of 8 so that as many
// loads are in flight per thread (populations read from global memory are
// latency-bound otherwise); the one-wave kernel reads LDS and keeps one.
template <int NT, typename K, typename KeyFn, typename Fn>
__device__ __forceinline__ void for_keys(int64_t count, KeyFn key, Fn fn) {
  constexpr int B = NT >= 256 ? 8 : 1;
  int64_t i = threadIdx.x;
  if constexpr (B > 1) {
    for (; i + (int64_t)(B - 1) * NT < count; i += (int64_t)B * NT) {
      K kv[B];
#pragma unroll
      for (int u = 0; u < B; ++u) kv[u] = key(i + (int64_t)u * NT);
#pragma unroll
      for (int u = 0; u < B; ++u) fn(i + (int64_t)u * NT, kv[u]);
    }
  }
  for (; i < count; i += NT) fn(i, key(i));
}

struct SelScratch {
  unsigned* hist;            // 2^DB bins
  unsigned* wsum;            // NT / 64
  unsigned long long* sh;    // 4
  unsigned long long* red;   // 2 * NT / 64
  unsigned long long* cand;  // SEL_CAND
  unsigned* ncand;           // 1
  float* comp;               // compacted values still in play (LDS), comp_cap of them
  int64_t comp_cap;          // 0: no compaction
};

// Appends v to sc.comp where hit, one LDS atomic per wave: the lanes that
// hit take consecutive slots after the count so far.
__device__ __forceinline__ void append_wave(const SelScratch& sc, bool hit, float v) {
  const unsigned long long bal = __ballot(hit);
  if (bal == 0ull) return;
  const int lane = (int)(threadIdx.x & 63u);
  const int leader = __ffsll((long long)bal) - 1;
  unsigned base = 0u;
  if (lane == leader) base = atomicAdd(sc.ncand, (unsigned)__popcll(bal));
  base = __shfl(base, leader);
  if (hit) sc.comp[base + (unsigned)__popcll(bal & ((1ull << lane) - 1ull))] = v;
}

// k-th smallest (0-based) key of the population, most significant digit
// first, for keys known to lie in [kmin, kmax].  Element i has the value
// VAL(i) and the unsigned key KEYOF(value).  Bits that every key in the
// range shares need no pass.  Once the digit that holds rank k has at most
// comp_cap keys, one pass copies their values into sc.comp and every later
// pass scans only those.  When it has at most SEL_CAND keys, one pass
// gathers them and one wave ranks them.  With want2, the key of rank k+1 is
// also returned (has2) when it lies among the same candidates.
template <int NT, int DB, typename K, typename ValFn, typename KeyOf>
__device__ __forceinline__ K radix_select(int64_t count, int64_t k, K kmin, K kmax, ValFn val, KeyOf keyof,
                          const SelScratch& sc, bool want2, K& v2, bool& has2) {
  constexpr int W = (int)sizeof(K) * 8;
  constexpr int NBINS = 1 << DB;
  has2 = false;
  // the range and counts are block-uniform; say so to the compiler, so the
  // pass loop below (barriers inside) is a scalar loop
  if constexpr (sizeof(K) == 8) {
    kmin = (K)rfl64((int64_t)kmin);
    kmax = (K)rfl64((int64_t)kmax);
  } else {
    kmin = (K)__builtin_amdgcn_readfirstlane((int)kmin);
    kmax = (K)__builtin_amdgcn_readfirstlane((int)kmax);
  }
  count = rfl64(count);
  k = rfl64(k);
  const K diff = kmin ^ kmax;
  if (diff == 0) {  // every key equals kmin
    v2 = kmin;
    has2 = true;
    return kmin;
  }
  int top = W - 1;  // highest differing bit
  while (!((diff >> top) & (K)1)) --top;
  top = __builtin_amdgcn_readfirstlane(top);
  const K low = (top + 1 >= W) ? ~(K)0 : (((K)1 << (top + 1)) - 1);
  K prefix = kmin & ~low, mask = ~low;
  int64_t kk = k;
  // keys scanned per pass: the whole population, or its compacted part
  bool compact = false;
  int64_t n_in = count;
  auto key = [&](int64_t i) -> K { return compact ? keyof(sc.comp[i]) : keyof(val(i)); };
  for (int hi = top + 1; hi > 0; hi -= DB) {
    const int width = hi >= DB ? DB : hi;
    const int shift = hi - width;
    const K dmask = (K)((1u << width) - 1u);
    for (int i = threadIdx.x; i < NBINS; i += NT) sc.hist[i] = 0;
    __syncthreads();
    for_keys<NT, K>(n_in, key, [&](int64_t, K kv) {
      if ((kv & mask) == prefix) atomicAdd(&sc.hist[(unsigned)((kv >> shift) & dmask)], 1u);
    });
    __syncthreads();
    find_digit<NT, NBINS>(sc.hist, kk, sc.wsum, sc.sh);
    // block-uniform values read back from LDS: made wave-uniform, so that
    // the branches and loop exits that depend on them are scalar
    const unsigned digit = (unsigned)__builtin_amdgcn_readfirstlane((int)sc.sh[0]);
    int64_t c = (int64_t)(unsigned)__builtin_amdgcn_readfirstlane((int)sc.hist[digit]);  // keys sharing the extended prefix
    prefix |= (K)digit << shift;
    mask |= dmask << shift;
    kk = rfl64((int64_t)sc.sh[1]);
    __syncthreads();
    if (shift == 0) {  // all bits resolved: the key is the prefix, repeated c times
      if (want2 && kk + 1 < c) {
        v2 = prefix;
        has2 = true;
      }
      return prefix;
    }
    if (c <= SEL_CAND) {
      // With rank k the largest key of its digit, rank k+1 is the smallest
      // key of the next non-empty digit of this pass: gather that digit
      // too when both fit.
      K prefix2 = prefix;
      int64_t c2 = 0;
      if (want2 && kk + 1 == c) {
        if (threadIdx.x == 0) *sc.ncand = NBINS;
        __syncthreads();
        for (int b = (int)digit + 1 + threadIdx.x; b < NBINS; b += NT)
          if (sc.hist[b] != 0u) atomicMin(sc.ncand, (unsigned)b);
        __syncthreads();
        const unsigned d2 = (unsigned)__builtin_amdgcn_readfirstlane((int)*sc.ncand);
        if (d2 < (unsigned)NBINS && c + (int64_t)sc.hist[d2] <= SEL_CAND) {
          prefix2 = (prefix & ~(dmask << shift)) | ((K)d2 << shift);
          c2 = sc.hist[d2];
        }
        __syncthreads();
      }
      if (threadIdx.x == 0) *sc.ncand = 0;
      __syncthreads();
      for_keys<NT, K>(n_in, key, [&](int64_t, K kv) {
        const K km = kv & mask;
        if (km == prefix || (c2 > 0 && km == prefix2))
          sc.cand[atomicAdd(sc.ncand, 1u)] = (unsigned long long)kv;
      });
      c += c2;
      __syncthreads();
      if (threadIdx.x < 64) {
        const int lane = threadIdx.x;
        const K mine = lane < c ? (K)sc.cand[lane] : ~(K)0;
        int64_t less = 0, same = 0;
        for (int t = 0; t < (int)c; ++t) {
          const K o = (K)sc.cand[t];
          less += o < mine;
          same += o == mine;
        }
        // a lane whose key covers rank kk (ties write the same value)
        if (lane < c && less <= kk && kk < less + same) sc.sh[2] = (unsigned long long)mine;
        if (lane < c && less <= kk + 1 && kk + 1 < less + same) sc.sh[3] = (unsigned long long)mine;
      }
      __syncthreads();
      const K v1 = (K)sc.sh[2];
      if (want2 && kk + 1 < c) {
        v2 = (K)sc.sh[3];
        has2 = true;
      }
      __syncthreads();
      return v1;
    }
    if (!compact && c <= sc.comp_cap) {
      // the c keys sharing the prefix: their values into sc.comp (in any
      // order; only counts and values matter from here on)
      if (threadIdx.x == 0) *sc.ncand = 0;
      __syncthreads();
      for_keys<NT, float>(n_in, val, [&](int64_t, float v) {
        append_wave(sc, (keyof(v) & mask) == prefix, v);
      });
      __syncthreads();
      compact = true;
      n_in = c;
    }
  }
  return prefix;  // not reached: the last pass has shift == 0
}

// Ascending bitonic sort of one key per lane across a wave (64 keys), by
// cross-lane exchanges: no LDS, no block barrier.
template <typename K>
__device__ __forceinline__ K wave_sort64(K v) {
  const int lane = (int)(threadIdx.x & 63u);
#pragma unroll
  for (int k = 2; k <= 64; k <<= 1) {
#pragma unroll
    for (int j = k >> 1; j > 0; j >>= 1) {
      K o;
      if constexpr (sizeof(K) == 8) {
        o = (K)__shfl_xor((unsigned long long)v, j);
      } else {
        o = (K)__shfl_xor((unsigned)v, j);
      }
      const bool lower = (lane & j) == 0;        // keeps the smaller of the pair
      const bool up = (lane & k) == 0;           // ascending run
      const K mn = o < v ? o : v, mx = o < v ? v : o;
      v = (lower == up) ? mn : mx;
    }
  }
  return v;
}

// Exact k-th smallest key (and the (k+1)-th when it sits in the same or
// the next non-empty bin, has2) with bins fitted to the data.  The range
// [kmin, kmax] that the radix passes split is set by the extreme keys, and
// when a few outliers stretch it, the first digit puts the bulk of the keys
// into a handful of bins, whose LDS atomics then serialise.  Here wave 0
// sorts a 64-key sample (odd stride) in registers and takes the window
// [lo, hi] between its ranks 8 and 56; one pass histograms every key into
// NBINS - 2 equal bins of 2^s keys across the window plus an underflow and
// an overflow bin, and when the bin holding rank k has at most SEL_CAND
// keys, one pass gathers them and one wave ranks them.  Returns false with
// nothing selected when rank k falls outside the window or its bin holds
// more keys (the caller then runs the radix selection).
template <int NT, int NBINS, typename K, typename ValFn, typename KeyOf>
__device__ __forceinline__ bool window_select(int64_t n, int64_t k, bool want2, ValFn val, KeyOf keyof,
                                              const SelScratch& sc, K& v1, K& v2, bool& has2) {
  const int lane = (int)(threadIdx.x & 63u);
  auto key = [&](int64_t i) -> K { return keyof(val(i)); };
  has2 = false;
  if (threadIdx.x < 64) {
    int64_t stride = n / 64;
    if (stride % 2 == 0) --stride;
    const K srt = wave_sort64<K>(key((int64_t)lane * stride));
    K lo, hi;
    if constexpr (sizeof(K) == 8) {
      lo = (K)__shfl((unsigned long long)srt, 8);
      hi = (K)__shfl((unsigned long long)srt, 56);
    } else {
      lo = (K)__shfl((unsigned)srt, 8);
      hi = (K)__shfl((unsigned)srt, 56);
    }
    int sh = 0;
    while (sh < (int)(8 * sizeof(K)) - 1 && ((hi - lo) >> sh) >= (K)(NBINS - 2)) ++sh;
    if (lane == 0) {
      sc.sh[0] = (unsigned long long)lo;
      sc.sh[1] = (unsigned long long)sh;
    }
  }
  for (int i = threadIdx.x; i < NBINS; i += NT) sc.hist[i] = 0;
  __syncthreads();
  const K lo = (K)rfl64((int64_t)sc.sh[0]);
  const int sh = __builtin_amdgcn_readfirstlane((int)sc.sh[1]);
  auto bin = [&](K kv) -> unsigned {
    if (kv < lo) return 0u;
    const K q = (kv - lo) >> sh;
    return q >= (K)(NBINS - 2) ? (unsigned)(NBINS - 1) : (unsigned)q + 1u;
  };
  __syncthreads();  // lo and sh read before sh[] is reused
  // keys outside the window all land in the two end bins: counted in
  // registers and added once per wave instead of by same-address atomics
  // (32-bit keys; with 64-bit keys the extra tests cost more VALU time
  // than the atomics they save)
  if constexpr (sizeof(K) == 4) {
    unsigned under = 0u, over = 0u;
    for_keys<NT, K>(n, key, [&](int64_t, K kv) {
      const unsigned q = bin(kv);
      if (q == 0u) ++under;
      else if (q == (unsigned)(NBINS - 1)) ++over;
      else atomicAdd(&sc.hist[q], 1u);
    });
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
      under += __shfl_xor(under, d);
      over += __shfl_xor(over, d);
    }
    if (lane == 0) {
      if (under) atomicAdd(&sc.hist[0], under);
      if (over) atomicAdd(&sc.hist[NBINS - 1], over);
    }
  } else {
    for_keys<NT, K>(n, key, [&](int64_t, K kv) { atomicAdd(&sc.hist[bin(kv)], 1u); });
  }
  __syncthreads();
  find_digit<NT, NBINS>(sc.hist, k, sc.wsum, sc.sh);
  const unsigned b = (unsigned)__builtin_amdgcn_readfirstlane((int)sc.sh[0]);
  const int64_t kk = rfl64((int64_t)sc.sh[1]);
  int64_t c = (int64_t)(unsigned)__builtin_amdgcn_readfirstlane((int)sc.hist[b]);
  __syncthreads();
  if (b == 0u || b == (unsigned)(NBINS - 1) || (c > SEL_CAND && c > sc.comp_cap)) return false;
  if (c > SEL_CAND) {
    // a fuller bin: its values into the compaction buffer, then the radix
    // selection among them, within the bin's key range
    if (threadIdx.x == 0) *sc.ncand = 0;
    __syncthreads();
    for_keys<NT, float>(n, val, [&](int64_t, float v) { append_wave(sc, bin(keyof(v)) == b, v); });
    __syncthreads();
    const K base = (K)(b - 1u) << sh;
    const K kmin = lo + base;
    const K span = (K)1 << sh;
    const K kmax = kmin + (span - 1) < kmin ? ~(K)0 : kmin + (span - 1);
    SelScratch in = sc;
    in.comp_cap = 0;
    const float* cv = sc.comp;
    auto cval = [&](int64_t i) -> float { return cv[i]; };
    v1 = radix_select<NT, NBINS == 2048 ? 11 : 8, K>(c, kk, kmin, kmax, cval, keyof, in, want2, v2, has2);
    return true;
  }
  // with rank k the last key of its bin, rank k+1 is the smallest key of the
  // next non-empty bin: gather that bin too when it is an interior one and fits
  unsigned b2 = (unsigned)NBINS;
  if (want2 && kk + 1 == c) {
    if (threadIdx.x == 0) *sc.ncand = (unsigned)NBINS;
    __syncthreads();
    for (int q = (int)b + 1 + threadIdx.x; q < NBINS; q += NT)
      if (sc.hist[q] != 0u) atomicMin(sc.ncand, (unsigned)q);
    __syncthreads();
    const unsigned d2 = (unsigned)__builtin_amdgcn_readfirstlane((int)*sc.ncand);
    if (d2 < (unsigned)(NBINS - 1) && c + (int64_t)sc.hist[d2] <= SEL_CAND) b2 = d2;
    __syncthreads();
  }
  const int64_t c2 = b2 < (unsigned)NBINS ? (int64_t)sc.hist[b2] : 0;
  if (threadIdx.x == 0) *sc.ncand = 0;
  __syncthreads();
  for_keys<NT, K>(n, key, [&](int64_t, K kv) {
    const unsigned q = bin(kv);
    if (q == b || q == b2) sc.cand[atomicAdd(sc.ncand, 1u)] = (unsigned long long)kv;
  });
  c += c2;
  __syncthreads();
  if (threadIdx.x < 64) {
    // rank every candidate against the others, held one per lane
    const K mine = lane < c ? (K)sc.cand[lane] : ~(K)0;
    int64_t less = 0, same = 0;
    for (int t = 0; t < (int)c; ++t) {
      K o;
      if constexpr (sizeof(K) == 8) {
        const uint32_t olo = __builtin_amdgcn_readlane((uint32_t)mine, t);
        const uint32_t ohi = __builtin_amdgcn_readlane((uint32_t)(mine >> 32), t);
        o = (K)(((uint64_t)ohi << 32) | olo);
      } else {
        o = (K)__builtin_amdgcn_readlane((uint32_t)mine, t);
      }
      less += o < mine;
      same += o == mine;
    }
    if (lane < c && less <= kk && kk < less + same) sc.sh[2] = (unsigned long long)mine;
    if (lane < c && less <= kk + 1 && kk + 1 < less + same) sc.sh[3] = (unsigned long long)mine;
  }
  __syncthreads();
  v1 = (K)sc.sh[2];
  if (want2 && kk + 1 < c) {
    v2 = (K)sc.sh[3];
    has2 = true;
  }
  __syncthreads();
  return true;
}

// The order statistic of rank k+1 given the one of rank k (key kk): kk
// itself if more than k+1 keys are <= kk, else the smallest key above kk.
// One pass: a count and a minimum, reduced over the block.
template <int NT, typename K, typename KeyFn>
__device__ __forceinline__ K next_rank(int64_t count, int64_t k, K kk, KeyFn key, unsigned long long* red) {
  constexpr int NW = NT / 64;
  unsigned long long le = 0;
  K mn = ~(K)0;
  for_keys<NT, K>(count, key, [&](int64_t, K kv) {
    if (kv <= kk) ++le;
    else if (kv < mn) mn = kv;
  });
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) {
    le += __shfl_down(le, d);
    const K o = (K)__shfl_down((unsigned long long)mn, d);
    mn = o < mn ? o : mn;
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) {
    red[2 * wave] = le;
    red[2 * wave + 1] = (unsigned long long)mn;
  }
  __syncthreads();
  unsigned long long tle = 0;
  K tmn = ~(K)0;
  for (int w = 0; w < NW; ++w) {
    tle += red[2 * w];
    const K o = (K)red[2 * w + 1];
    tmn = o < tmn ? o : tmn;
  }
  __syncthreads();
  return (int64_t)tle > k + 1 ? kk : tmn;
}

__device__ __forceinline__ Pop make_pop(int64_t id, int64_t n_time, int64_t n_base, int n_chan,
                                        int population) {
  const int64_t plane = n_base * (int64_t)n_chan;
  if (population == 0) return Pop{id * n_chan, n_time * n_chan, n_chan, 1, plane};
  if (population == 1) {
    const int64_t b = id / n_chan, k = id % n_chan;
    return Pop{b * n_chan + k, n_time, 1, 0, plane};
  }
  const int64_t t = id / n_base, b = id % n_base;
  return Pop{t * plane + b * n_chan, n_chan, n_chan, 1, 0};
}

}  // namespace

// One block per population.  Amplitudes are cached in dynamic LDS when the
// population has at most `cap` members.
// Amplitudes of every population, each population contiguous:
// amp[id * count + i] = |V| of its element i (as amp_f32).
__global__ void mad_amp_kernel(const float2* __restrict__ vis, int64_t n_time, int64_t n_base, int n_chan,
                               int population, int64_t count, int64_t total, float* __restrict__ amp) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= total) return;
  int64_t id, i;
  if (total <= 0x7fffffffLL) {  // 32-bit division
    const uint32_t q = (uint32_t)e / (uint32_t)count;
    id = q;
    i = (uint32_t)e - q * (uint32_t)count;
  } else {
    id = e / count;
    i = e % count;
  }
  amp[e] = amp_f32(vis[make_pop(id, n_time, n_base, n_chan, population).off(i)]);
}

// The same for per-baseline populations (contiguous runs of n_chan, a
// multiple of 4) of a 32-byte aligned plane: four amplitudes per thread from
// two 16-byte loads, written with one 16-byte store.
__global__ void mad_amp4_kernel(const float4* __restrict__ vis, int64_t n_base, int n_chan, int64_t count,
                                int64_t total4, float4* __restrict__ amp) {
  const int64_t e4 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e4 >= total4) return;
  const int64_t e = 4 * e4;
  int64_t id, t, k;  // baseline, integration, channel (k % 4 == 0)
  if (4 * total4 <= 0x7fffffffLL) {  // 32-bit division
    const uint32_t q = (uint32_t)e / (uint32_t)count, i = (uint32_t)e - q * (uint32_t)count;
    const uint32_t tq = i / (uint32_t)n_chan;
    id = q;
    t = tq;
    k = i - tq * (uint32_t)n_chan;
  } else {
    const int64_t i = e % count;
    id = e / count;
    t = i / n_chan;
    k = i % n_chan;
  }
  const int64_t v = ((t * n_base + id) * n_chan + k) / 2;  // float4 = two visibilities
  const float4 a = vis[v], b = vis[v + 1];
  amp[e4] = make_float4(amp_f32(make_float2(a.x, a.y)), amp_f32(make_float2(a.z, a.w)),
                        amp_f32(make_float2(b.x, b.y)), amp_f32(make_float2(b.z, b.w)));
}

// ---- large populations: one pass over the visibilities ---------------------
//
// A population's median, MAD and flags take one read of its visibilities when
// a sample says beforehand where the median, the MAD and the threshold lie:
//   1. mad_sample_kernel, a workgroup per population: amplitudes of MAD_SAMPLE
//      elements (jittered strata of four neighbours) bound the median in
//      [lo, hi] and the MAD in [dlo, dhi];
//   2. mad_scan_kernel, the whole GPU: counts the amplitudes below the median's
//      window, keeps those inside it; keeps the amplitudes whose deviation
//      from some median in [lo, hi] can lie in [dlo, dhi] and counts those
//      whose deviation cannot exceed dlo; writes the flags that any threshold
//      in [lo + c dlo, hi + c dhi] decides alike and keeps the others;
//   3. mad_finish_kernel, a workgroup per population: exact selection among the
//      kept amplitudes at the ranks the counts leave, the threshold, the
//      remaining flags.
// Ranks and counts are of the whole population, so the results are the exact
// order statistics.  A population that the sample cannot bound (half of it zero)
// or whose lists would overflow (large groups of equal amplitudes) is open from
// step 1: step 2 then forms its amplitudes, over its lists, and mad_kernel
// selects among those from the start.  One whose rank falls outside its window
// all the same (a sample that misled) stays at MAD_SCAN; mad_kernel forms the
// amplitudes on its first pass.
// 528 planes of 524288, all open because half of each is zero: 10.7 ms, 10.6
// without the sample (18.1 ms with the amplitudes formed anew by every pass of
// mad_kernel); of amplitudes that repeat: 5.2 ms (15.7).
//
// Bound: HBM, 8 B a visibility read and 1 B written, and the scan's vector
// instructions beside it.  528 planes of 524288 visibilities: 0.82 ms (sample
// 0.06, scan 0.65 = 4.2 TB/s with the lists, finish 0.15); 2.45 ms with the amplitudes
// written out first and a workgroup per population selecting among them.
enum { MAD_OPEN = 0, MAD_SCAN = 1, MAD_DONE = 2 };
struct MadWin {
  int state;
  float lo, hi;                  // the median lies in (lo, hi)
  float q_lo, q_hi;              // their squares, and those of
  float q_l0, q_c0, q_c1, q_r1;  //   l0 < c0 < lo < hi < c1 < r1: amplitudes outside [l0, r1] deviate
                                 //   by dhi or more, those inside [c0, c1] by dlo or less
  float q_t0, q_t1;              //   and t0, t1: T lies in [t0, t1]
  float r1;
  uint32_t n_le, n_in;           // amplitudes up to lo; inside [c0, c1]
  uint32_t n_med, n_dev, n_thr;  // entries of the three lists (also past their capacity)
  double dlo, dhi;
};

// The scan compares float32 squares |V|^2 with the windows' squares, not the
// amplitudes: what it takes for a <= x has a <= x (1 + MAD_EPS), and likewise
// the other way round (rounding of both squares: 3 2^-24 of the amplitude).
// The finish accepts a result only if it keeps that distance from its window.
constexpr double MAD_EPS = 4e-7;

constexpr int MAD_SAMPLE_NT = 512;
constexpr int MAD_SAMPLE_PER = 24;
constexpr int MAD_SAMPLE = MAD_SAMPLE_NT * MAD_SAMPLE_PER;  // 12288
constexpr int MAD_SLACK = 333;       // ranks of the sample on each side: 6 standard deviations of its median's
constexpr int MAD_CHUNK = 16384;     // elements per scan workgroup

// Capacities of the three lists of a population of n: about 5 % and 13 % of a
// smooth population fall to the first two.
__host__ __device__ __forceinline__ int64_t mad_cap_med(int64_t n) { return n / 8; }
__host__ __device__ __forceinline__ int64_t mad_cap_dev(int64_t n) { return n / 4; }
__host__ __device__ __forceinline__ int64_t mad_cap_thr(int64_t n) { return n / 16; }
// The lists of one population lie in the first half of its n floats, which its
// amplitudes take if it is left open.

// The four amplitudes at elements i..i+3 of a population (i % 4 == 0).  VEC:
// rows are multiples of four elements and 16-byte aligned.
template <bool VEC>
__device__ __forceinline__ void amp4(const float2* __restrict__ vis, const Pop& pop, int64_t i, float a[4]) {
  if constexpr (VEC) {
    const float4* p = reinterpret_cast<const float4*>(vis + pop.off(i));
    const float4 u = p[0], v = p[1];
    a[0] = amp_f32(make_float2(u.x, u.y)), a[1] = amp_f32(make_float2(u.z, u.w));
    a[2] = amp_f32(make_float2(v.x, v.y)), a[3] = amp_f32(make_float2(v.z, v.w));
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j) a[j] = amp_f32(vis[pop.off(i + j)]);
  }
}

// Bounds of the sample's order statistics of ranks MAD_SAMPLE/2 -+ MAD_SLACK
// over keys kv[] (16 per thread): the edges of their bins in a histogram over
// the middle three quarters of a 64-key subsample.  False when a rank falls
// outside it, or when more than `most` of the sample lie within the bounds.
__device__ __forceinline__ bool sample_bounds(const float (&a)[MAD_SAMPLE_PER], float centre, unsigned* hist,
                                              unsigned* wsum, unsigned long long* sh, unsigned* sub, unsigned most,
                                              uint32_t& klo, uint32_t& khi) {
  constexpr int NT = MAD_SAMPLE_NT, NBINS = 2048;
  const int t = threadIdx.x;
  auto key = [&](int j) -> uint32_t { return __float_as_uint(fabsf(a[j] - centre)); };
  if (t % (NT / 64) == 0) sub[t / (NT / 64)] = key(5);
  for (int i = t; i < NBINS; i += NT) hist[i] = 0;
  __syncthreads();
  if (t < 64) {
    const uint32_t srt = wave_sort64<uint32_t>(sub[t]);
    const uint32_t lo = __shfl(srt, 8), hi = __shfl(srt, 56);
    int s = 0;
    while (s < 31 && ((hi - lo) >> s) >= (uint32_t)(NBINS - 2)) ++s;
    if (t == 0) {
      sh[2] = lo;
      sh[3] = (unsigned long long)s;
    }
  }
  __syncthreads();
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)sh[2]);
  const int s = __builtin_amdgcn_readfirstlane((int)sh[3]);
  unsigned under = 0u, over = 0u;
#pragma unroll
  for (int j = 0; j < MAD_SAMPLE_PER; ++j) {
    const uint32_t k = key(j), q = (k - lo) >> s;
    if (k < lo) ++under;
    else if (q >= (uint32_t)(NBINS - 2)) ++over;
    else atomicAdd(&hist[q + 1u], 1u);
  }
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) {
    under += __shfl_xor(under, d);
    over += __shfl_xor(over, d);
  }
  if ((t & 63) == 0) {
    if (under) atomicAdd(&hist[0], under);
    if (over) atomicAdd(&hist[NBINS - 1], over);
  }
  __syncthreads();
  find_digit<NT, NBINS>(hist, MAD_SAMPLE / 2 - MAD_SLACK, wsum, sh);
  const unsigned b0 = (unsigned)__builtin_amdgcn_readfirstlane((int)sh[0]);
  const unsigned in0 = (unsigned)__builtin_amdgcn_readfirstlane((int)sh[1]);  // of its bin, before the rank
  __syncthreads();
  find_digit<NT, NBINS>(hist, MAD_SAMPLE / 2 + MAD_SLACK, wsum, sh);
  const unsigned b1 = (unsigned)__builtin_amdgcn_readfirstlane((int)sh[0]);
  const unsigned in1 = (unsigned)__builtin_amdgcn_readfirstlane((int)sh[1]);
  const unsigned inside = in0 + 2 * MAD_SLACK + ((unsigned)__builtin_amdgcn_readfirstlane((int)hist[b1]) - in1);
  __syncthreads();
  if (b0 == 0u || b1 == (unsigned)(NBINS - 1) || inside > most) return false;
  klo = lo + ((b0 - 1u) << s);
  khi = lo + (b1 << s);
  return true;
}

template <bool VEC>
__global__ void __launch_bounds__(MAD_SAMPLE_NT)
mad_sample_kernel(const float2* __restrict__ vis, int64_t n_time, int64_t n_base, int n_chan, float sigma,
                  int population, MadWin* __restrict__ win) {
  __shared__ unsigned hist[2048];
  __shared__ unsigned wsum[MAD_SAMPLE_NT / 64];
  __shared__ unsigned long long sh[4];
  __shared__ unsigned sub[64];
  const Pop pop = make_pop(blockIdx.x, n_time, n_base, n_chan, population);
  const int64_t n4 = pop.count / 4;
  // strata of the population in order, four neighbouring elements of each,
  // their place in it scattered so that no channel or integration is favoured
  constexpr int STRATA = MAD_SAMPLE / 4, PER = MAD_SAMPLE_PER / 4;
  float a[MAD_SAMPLE_PER];
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int64_t g = PER * (int64_t)threadIdx.x + q;
    const int64_t g0 = g * n4 / STRATA, g1 = (g + 1) * n4 / STRATA;
    const uint32_t h = ((uint32_t)g * 2654435761u) >> 8;
    amp4<VEC>(vis, pop, 4 * (g0 + (int64_t)(h % (uint32_t)(g1 - g0))), a + 4 * q);
  }
  uint32_t k0 = 0u, k1 = 0u, e0 = 0u, e1 = 0u;
  // the median's list takes an eighth of the population; the deviations' a
  // quarter, of which the slack added below takes about 8 %
  bool ok = sample_bounds(a, 0.f, hist, wsum, sh, sub, MAD_SAMPLE / 8, k0, k1);
  const float lo = __uint_as_float(k0), hi = __uint_as_float(k1);
  // the sample's deviations are from the centre of the median's window
  if (ok) ok = sample_bounds(a, 0.5f * (lo + hi), hist, wsum, sh, sub, MAD_SAMPLE / 6, e0, e1);
  if (threadIdx.x != 0) return;
  MadWin w;
  w.state = MAD_OPEN;
  w.n_le = w.n_in = w.n_med = w.n_dev = w.n_thr = 0u;
  if (ok) {
    // a quarter of the median's window covers what the true median moves the
    // MAD by
    const double slack = 0.25 * ((double)hi - (double)lo) + 4.0 * MAD_EPS * hi;
    w.lo = lo;
    w.hi = hi;
    w.dlo = (double)__uint_as_float(e0) - slack;
    w.dhi = (double)__uint_as_float(e1) + slack;
    const double c = (double)sigma * 1.4826;
    const float t0 = (float)((lo + c * w.dlo) * (1.0 - 4.0 * MAD_EPS));
    const float t1 = (float)((hi + c * w.dhi) * (1.0 + 4.0 * MAD_EPS));
    const float l0 = (float)((double)lo - w.dhi), c0 = (float)((double)hi - w.dlo);
    const float c1 = (float)((double)lo + w.dlo), r1 = (float)((double)hi + w.dhi);
    // an upper or lower band can be empty (the MAD exceeds the median):
    // negative bounds have no amplitude below them
    auto sq = [](float v) -> float { return v < 0.f ? -1.f : v * v; };
    w.r1 = r1;
    w.q_lo = sq(lo);
    w.q_hi = sq(hi);
    w.q_l0 = sq(l0);
    w.q_c0 = sq(c0);
    w.q_c1 = sq(c1);
    w.q_r1 = sq(r1);
    w.q_t0 = sq(t0);
    w.q_t1 = sq(t1);
    // the windows in order, and every square a normal float32
    if (c0 < lo && hi < c1 && lo > 1e-15f && r1 < 1e18f && t1 < 1e18f) w.state = MAD_SCAN;
  }
  win[blockIdx.x] = w;
}

constexpr int MAD_SCAN_LIST = 640;  // per wave; 256 entries at most come between flushes

template <bool VEC>
__global__ void __launch_bounds__(256)
mad_scan_kernel(const float2* __restrict__ vis, int64_t n_time, int64_t n_base, int n_chan, int population,
                int chunks, MadWin* __restrict__ win, float* __restrict__ lists, uint8_t* __restrict__ mask) {
  constexpr int NT = 256;
  // each wave keeps a list of its own: appending needs no atomics
  __shared__ float2 list_l[NT / 64][MAD_SCAN_LIST];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t id = blockIdx.x / (unsigned)chunks;
  const int64_t i0 = (int64_t)(blockIdx.x % (unsigned)chunks) * MAD_CHUNK;
  MadWin* const w = win + id;
  const Pop pop = make_pop(id, n_time, n_base, n_chan, population);
  const int64_t n = pop.count;
  if (w->state != MAD_SCAN) {  // open: the chunk's amplitudes
    constexpr int U = 4;
    float* const o = lists + id * n;
    const int64_t end = i0 + MAD_CHUNK < n ? i0 + MAD_CHUNK : n;
    for (int64_t k0 = i0 + 4 * (int)threadIdx.x; k0 < end; k0 += 4 * U * NT) {
      float a[U][4];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t k = k0 + 4 * u * NT;
        if (VEC) {
          amp4<true>(vis, pop, k < end ? k : k0, a[u]);
        } else {
#pragma unroll
          for (int j = 0; j < 4; ++j) a[u][j] = amp_f32(vis[pop.off(k + j < end ? k + j : k0)]);
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t k = k0 + 4 * u * NT;
        if (VEC) {
          if (k < end) *reinterpret_cast<float4*>(o + k) = make_float4(a[u][0], a[u][1], a[u][2], a[u][3]);
        } else {
#pragma unroll
          for (int j = 0; j < 4; ++j)
            if (k + j < end) o[k + j] = a[u][j];
        }
      }
    }
    return;
  }
  float* const g_med = lists + id * n;
  float* const g_dev = g_med + mad_cap_med(n);
  float* const g_thr = g_dev + mad_cap_dev(n);
  const float q_lo = w->q_lo, q_hi = w->q_hi, q_l0 = w->q_l0, q_c0 = w->q_c0, q_c1 = w->q_c1, q_r1 = w->q_r1;
  const float q_t0 = mask ? w->q_t0 : __builtin_inff(), q_t1 = w->q_t1;
  float2* const list = list_l[wave];
  unsigned m = 0u;                  // wave-uniform
  unsigned n_le = 0u, n_in = 0u;    // per lane
  const unsigned long long below = (1ull << lane) - 1ull;
  auto square = [](float2 z) -> float { return z.x * z.x + z.y * z.y; };
  // the list's exact amplitudes to the population's two lists, in any order
  auto flush = [&]() {
    unsigned k_med = 0u;
    for (unsigned k = lane; k < m; k += 64) {
      const float sq = square(list[k]);
      k_med += !(sq <= q_lo) && sq <= q_hi;
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) k_med += __shfl_xor(k_med, d);
    unsigned at = 0u;
    if (lane < 2) at = atomicAdd(lane == 0 ? &w->n_med : &w->n_dev, lane == 0 ? k_med : m - k_med);
    unsigned at_m = __builtin_amdgcn_readlane(at, 0), at_d = __builtin_amdgcn_readlane(at, 1);
    for (unsigned k0 = 0u; k0 < m; k0 += 64) {
      const bool in = k0 + lane < m;
      const float2 z = list[in ? k0 + lane : 0];
      const float sq = square(z), a = amp_f32(z);
      const bool med = !(sq <= q_lo) && sq <= q_hi;
      const unsigned long long bm = __ballot(in && med), bd = __ballot(in && !med);
      const unsigned pm = at_m + (unsigned)__popcll(bm & below), pd = at_d + (unsigned)__popcll(bd & below);
      if (in && med && pm < (unsigned)mad_cap_med(n)) g_med[pm] = a;
      if (in && !med && pd < (unsigned)mad_cap_dev(n)) g_dev[pd] = a;
      at_m += (unsigned)__popcll(bm);
      at_d += (unsigned)__popcll(bd);
    }
    m = 0u;
  };
  // four neighbouring elements per thread and step, the next two steps' loads
  // in flight
  struct Step {
    float2 v[4];
    int64_t off;
  };
  auto load = [&](int64_t i) -> Step {
    Step s;
    if (VEC) {  // n is a multiple of four
      s.off = pop.off(i < n ? i : 0);
      const float4* p = reinterpret_cast<const float4*>(vis + s.off);
      const float4 x = p[0], y = p[1];
      s.v[0] = make_float2(x.x, x.y), s.v[1] = make_float2(x.z, x.w);
      s.v[2] = make_float2(y.x, y.y), s.v[3] = make_float2(y.z, y.w);
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) s.v[j] = vis[pop.off(i + j < n ? i + j : 0)];
    }
    return s;
  };
  const int64_t end = i0 + MAD_CHUNK < n ? i0 + MAD_CHUNK : n;
  int64_t i = i0 + 4 * (int)threadIdx.x;
  Step s0 = load(i), s1 = load(i + 4 * NT);
#pragma unroll 1
  for (int64_t b0 = i0; b0 < end; b0 += 4 * NT, i += 4 * NT) {
    const Step s = s0;
    s0 = s1;
    s1 = load(i + 8 * NT);
    if (m > MAD_SCAN_LIST - 4 * 64) flush();
    bool over = false;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float sq = square(s.v[j]);
      // tests that a NaN passes: it stands above every amplitude
      const bool in = VEC ? i < n : i + j < n;
      const bool p_c0 = !(sq < q_c0), p_lo = !(sq <= q_lo), p_c1 = !(sq <= q_c1);
      n_le += in && !p_lo;
      n_in += in && p_c0 && !p_c1;
      over = over || !(sq <= q_t0);
      const unsigned long long hit =
          __ballot(in) & ((__ballot(!(sq < q_l0)) & ~__ballot(p_c0)) | (__ballot(p_lo) & ~__ballot(!(sq <= q_hi))) |
                          (__ballot(p_c1) & ~__ballot(!(sq <= q_r1))));
      if (hit != 0ull) {
        if ((hit >> lane) & 1ull) list[m + (unsigned)__popcll(hit & below)] = s.v[j];
        m += (unsigned)__popcll(hit);
      }
    }
    // flags: few amplitudes are over t0, and of those few under t1
    if (mask) {
      uint32_t flags = 0u;
      if (over) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float sq = square(s.v[j]);
          if (sq > q_t1) {
            flags |= 1u << (8 * j);
          } else if (i + j < n && !(sq <= q_t0)) {
            const unsigned k = atomicAdd(&w->n_thr, 1u);
            if (k < (unsigned)mad_cap_thr(n)) {
              g_thr[2 * (int64_t)k] = __uint_as_float((uint32_t)(i + j));
              g_thr[2 * (int64_t)k + 1] = amp_f32(s.v[j]);
            }
          }
        }
      }
      if (VEC) {
        if (i < n) *reinterpret_cast<uint32_t*>(mask + s.off) = flags;
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (i + j < n) mask[pop.off(i + j)] = (uint8_t)(flags >> (8 * j));
      }
    }
  }
  flush();
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) {
    n_le += __shfl_xor(n_le, d);
    n_in += __shfl_xor(n_in, d);
  }
  if (lane < 2) atomicAdd(lane == 0 ? &w->n_le : &w->n_in, lane == 0 ? n_le : n_in);
}

constexpr int MAD_FINISH_COMP = 8192;

// 512 threads leave room for three populations per CU (768 in one round),
// 1024 halve the time of one where there are CUs enough for all.
template <int NT>
__global__ void __launch_bounds__(NT, NT == 512 ? 6 : 4)
mad_finish_kernel(int64_t n_time, int64_t n_base, int n_chan, float sigma, int population,
                  MadWin* __restrict__ win, const float* __restrict__ lists, uint8_t* __restrict__ mask,
                  double* __restrict__ thresh, double* __restrict__ stats) {
  constexpr int DB = 11;
  __shared__ unsigned hist[1 << DB];
  __shared__ unsigned wsum[NT / 64];
  __shared__ unsigned long long sh[4];
  __shared__ unsigned long long red[2 * (NT / 64)];
  __shared__ unsigned long long cand[SEL_CAND];
  __shared__ unsigned ncand;
  __shared__ float comp[MAD_FINISH_COMP];
  const SelScratch sc{hist, wsum, sh, red, cand, &ncand, comp, MAD_FINISH_COMP};
  MadWin* const w = win + blockIdx.x;
  auto uni = [](uint32_t v) -> uint32_t { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); };
  if (uni((uint32_t)w->state) != MAD_SCAN) return;
  const Pop pop = make_pop(blockIdx.x, n_time, n_base, n_chan, population);
  const int64_t n = pop.count;
  const float* const g_med = lists + (int64_t)blockIdx.x * n;
  const float* const g_dev = g_med + mad_cap_med(n);
  const float* const g_thr = g_dev + mad_cap_dev(n);
  const int64_t n_med = uni(w->n_med), n_dev = uni(w->n_dev), n_thr = uni(w->n_thr);
  if (n_med > mad_cap_med(n) || n_dev > mad_cap_dev(n) || n_thr > mad_cap_thr(n)) return;
  const int64_t k1 = (n - 1) / 2, k2 = n / 2;
  const bool two = k2 != k1;
  // the median among the keys of its window
  const int64_t km = k1 - (int64_t)uni(w->n_le);
  if (km < 0 || km + (k2 - k1) >= n_med) return;
  auto aval = [&](int64_t i) -> float { return g_med[i]; };
  auto akeyof = [](float a) -> uint32_t { return __float_as_uint(a); };
  auto akey = [&](int64_t i) -> uint32_t { return __float_as_uint(g_med[i]); };
  uint32_t a1 = 0u, a2 = 0u;
  bool has2;
  if (n_med < 64 || !window_select<NT, (1 << DB), uint32_t>(n_med, km, two, aval, akeyof, sc, a1, a2, has2))
    a1 = radix_select<NT, DB, uint32_t>(n_med, km, 0u, __float_as_uint(w->r1), aval, akeyof, sc, two, a2, has2);
  if (!two) a2 = a1;
  else if (!has2) a2 = next_rank<NT, uint32_t>(n_med, km, a1, akey, red);
  a1 = uni(a1);
  a2 = uni(a2);
  const double v1 = (double)__uint_as_float(a1), v2 = (double)__uint_as_float(a2);
  if (!(v1 > w->lo * (1.0 + MAD_EPS) && v2 < w->hi * (1.0 - MAD_EPS))) return;
  const double med = (v1 + v2) / 2.0;
  // the MAD among the deviations that can reach it
  const int64_t kd = k1 - (int64_t)uni(w->n_in);
  if (kd < 0 || kd + (k2 - k1) >= n_dev) return;
  auto dval = [&](int64_t i) -> float { return g_dev[i]; };
  auto dkeyof = [&](float a) -> uint64_t { return (uint64_t)__double_as_longlong(fabs((double)a - med)); };
  auto dkey = [&](int64_t i) -> uint64_t { return dkeyof(g_dev[i]); };
  // a band amplitude is at most r1 (1 + MAD_EPS), and a deviation no larger
  const uint64_t dmax = (uint64_t)__double_as_longlong(2.0 * (double)w->r1);
  uint64_t d1 = 0ull, d2 = 0ull;
  if (n_dev < 64 || !window_select<NT, (1 << DB), uint64_t>(n_dev, kd, two, dval, dkeyof, sc, d1, d2, has2))
    d1 = radix_select<NT, DB, uint64_t>(n_dev, kd, 0ull, dmax, dval, dkeyof, sc, two, d2, has2);
  if (!two) d2 = d1;
  else if (!has2) d2 = next_rank<NT, uint64_t>(n_dev, kd, d1, dkey, red);
  d1 = (uint64_t)rfl64((int64_t)d1);
  d2 = (uint64_t)rfl64((int64_t)d2);
  const double m1 = __longlong_as_double((long long)d1), m2 = __longlong_as_double((long long)d2);
  const double eps = 2.0 * MAD_EPS * (double)w->r1;
  if (!(m1 > w->dlo + eps && m2 < w->dhi - eps)) return;
  const double madv = (m1 + m2) / 2.0;
  const double c = (double)sigma * 1.4826;
  const double T = med + c * madv;
  if (mask)
    for (int64_t k = threadIdx.x; k < n_thr; k += NT)
      mask[pop.off((int64_t)__float_as_uint(g_thr[2 * k]))] = (double)g_thr[2 * k + 1] > T ? 1 : 0;
  if (threadIdx.x == 0) {
    w->state = MAD_DONE;
    if (thresh) thresh[blockIdx.x] = T;
    if (stats) {
      stats[2 * (int64_t)blockIdx.x] = med;
      stats[2 * (int64_t)blockIdx.x + 1] = madv;
    }
  }
}

template <int NT, int DB>
__global__ void __launch_bounds__(NT)
mad_kernel(const float2* __restrict__ vis, int64_t n_time, int64_t n_base, int n_chan, float sigma,
           int population, int64_t cap, int64_t comp_cap, float* __restrict__ gamp_big,
           const MadWin* __restrict__ win, uint8_t* __restrict__ mask, double* __restrict__ thresh,
           double* __restrict__ stats) {
  // the amplitudes are in gamp, or (MAD_SCAN) go there on the first pass; small
  // populations have neither
  constexpr bool BIG = NT >= 1024;
  float* const gamp = BIG ? gamp_big : nullptr;
  bool formed = BIG && gamp != nullptr;
  if (BIG && win) {
    const int state = __builtin_amdgcn_readfirstlane(win[blockIdx.x].state);
    if (state == MAD_DONE) return;
    formed = formed && state == MAD_OPEN;
  }
  __shared__ unsigned hist[1 << DB];
  __shared__ unsigned wsum[NT / 64];
  __shared__ unsigned long long sh[4];
  __shared__ unsigned long long red[2 * (NT / 64)];
  __shared__ unsigned long long cand[SEL_CAND];
  __shared__ unsigned ncand;
  extern __shared__ __align__(16) float acache[];  // [cap] amplitude cache, then [comp_cap] compaction buffer
  const int64_t id = blockIdx.x;
  const Pop pop = make_pop(id, n_time, n_base, n_chan, population);
  const int64_t n = pop.count;
  const bool cached = n <= cap;
  const SelScratch sc{hist, wsum, sh, red, cand, &ncand, acache + (cached ? n : 0), comp_cap};
  const AmpSrc amp{vis, pop, cached ? acache : (gamp ? gamp + id * n : nullptr)};
  // one pass: the amplitudes into the LDS cache (when they fit) and the
  // range of their keys
  uint32_t amin = ~0u, amax = 0u;
  const bool vec4 = gamp && cached && n % 4 == 0 && (reinterpret_cast<uintptr_t>(gamp + id * n) & 15u) == 0;
  if (vec4) {
    // four amplitudes per 16-byte load, eight loads in flight per thread
    constexpr int U = 8;
    const float4* g4 = reinterpret_cast<const float4*>(gamp + id * n);
    float4* c4 = reinterpret_cast<float4*>(acache);
    const int64_t n4 = n / 4;
    for (int64_t j0 = threadIdx.x; j0 < n4; j0 += (int64_t)U * NT) {
      float4 a[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t j = j0 + (int64_t)u * NT;
        a[u] = j < n4 ? g4[j] : make_float4(0.f, 0.f, 0.f, 0.f);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t j = j0 + (int64_t)u * NT;
        if (j < n4) {
          c4[j] = a[u];
          const uint32_t k4[4] = {__float_as_uint(a[u].x), __float_as_uint(a[u].y), __float_as_uint(a[u].z),
                                  __float_as_uint(a[u].w)};
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            amin = k4[v] < amin ? k4[v] : amin;
            amax = k4[v] > amax ? k4[v] : amax;
          }
        }
      }
    }
  } else {
    // eight loads in flight per thread before their amplitudes are formed
    constexpr int U = 8;
    for (int64_t i0 = threadIdx.x; i0 < n; i0 += (int64_t)U * NT) {
      float a[U];
      if (formed) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int64_t i = i0 + (int64_t)u * NT;
          a[u] = i < n ? gamp[id * n + i] : 0.f;
        }
      } else {
        float2 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int64_t i = i0 + (int64_t)u * NT;
          v[u] = i < n ? vis[pop.off(i)] : make_float2(0.f, 0.f);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) a[u] = amp_f32(v[u]);
        if (BIG && gamp)
#pragma unroll
          for (int u = 0; u < U; ++u)
            if (i0 + (int64_t)u * NT < n) gamp[id * n + i0 + (int64_t)u * NT] = a[u];
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t i = i0 + (int64_t)u * NT;
        if (i < n) {
          if (cached) acache[i] = a[u];
          const uint32_t kv = __float_as_uint(a[u]);
          amin = kv < amin ? kv : amin;
          amax = kv > amax ? kv : amax;
        }
      }
    }
  }
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) {
    const uint32_t a = __shfl_down(amin, d), b = __shfl_down(amax, d);
    amin = a < amin ? a : amin;
    amax = b > amax ? b : amax;
  }
  if ((threadIdx.x & 63) == 0) {
    red[2 * (threadIdx.x >> 6)] = amin;
    red[2 * (threadIdx.x >> 6) + 1] = amax;
  }
  __syncthreads();
  amin = ~0u;
  amax = 0u;
  for (int w = 0; w < NT / 64; ++w) {
    amin = (uint32_t)red[2 * w] < amin ? (uint32_t)red[2 * w] : amin;
    amax = (uint32_t)red[2 * w + 1] > amax ? (uint32_t)red[2 * w + 1] : amax;
  }
  // block-uniform values from LDS, and every value derived from them below
  // (the medians, the key ranges): wave-uniform for the compiler, so the
  // selection loops that depend on them are scalar loops
  amin = (uint32_t)__builtin_amdgcn_readfirstlane((int)amin);
  amax = (uint32_t)__builtin_amdgcn_readfirstlane((int)amax);
  __syncthreads();
  const int64_t k1 = (n - 1) / 2, k2 = n / 2;
  auto akeyof = [](float a) -> uint32_t { return __float_as_uint(a); };
  auto akey = [&](int64_t i) -> uint32_t { return akeyof(amp(i)); };
  uint32_t a2;
  bool has2;
  // windowed first pass for the large populations, radix passes otherwise
  // (or when the window misses)
  constexpr bool WIN = NT >= 1024;
  uint32_t a1 = 0u;
  if (!(WIN && window_select<NT, (1 << DB), uint32_t>(n, k1, k2 != k1, amp, akeyof, sc, a1, a2, has2)))
    a1 = radix_select<NT, DB, uint32_t>(n, k1, amin, amax, amp, akeyof, sc, k2 != k1, a2, has2);
  if (k2 == k1) a2 = a1;
  else if (!has2) a2 = next_rank<NT, uint32_t>(n, k1, a1, akey, red);
  a1 = (uint32_t)__builtin_amdgcn_readfirstlane((int)a1);
  a2 = (uint32_t)__builtin_amdgcn_readfirstlane((int)a2);
  const double med = ((double)__uint_as_float(a1) + (double)__uint_as_float(a2)) / 2.0;
  auto dkeyof = [&](float a) -> uint64_t { return (uint64_t)__double_as_longlong(fabs((double)a - med)); };
  auto dkey = [&](int64_t i) -> uint64_t { return dkeyof(amp(i)); };
  // deviations lie in [0, the larger deviation of the two extreme amplitudes]
  const double dlo = fabs((double)__uint_as_float(amin) - med);
  const double dhi = fabs((double)__uint_as_float(amax) - med);
  const uint64_t dmax = (uint64_t)__double_as_longlong(dlo > dhi ? dlo : dhi);
  uint64_t d2;
  uint64_t d1 = 0ull;
  if (!(WIN && window_select<NT, (1 << DB), uint64_t>(n, k1, k2 != k1, amp, dkeyof, sc, d1, d2, has2)))
    d1 = radix_select<NT, DB, uint64_t>(n, k1, 0ull, dmax, amp, dkeyof, sc, k2 != k1, d2, has2);
  if (k2 == k1) d2 = d1;
  else if (!has2) d2 = next_rank<NT, uint64_t>(n, k1, d1, dkey, red);
  d1 = (uint64_t)rfl64((int64_t)d1);
  d2 = (uint64_t)rfl64((int64_t)d2);
  const double madv =
      (__longlong_as_double((long long)d1) + __longlong_as_double((long long)d2)) / 2.0;
  const double c = (double)sigma * 1.4826;
  const double T = med + c * madv;
  if (mask) {
    if (cached && pop.s_inner == 1 && pop.inner_n % 4 == 0 && pop.base % 4 == 0 && pop.s_outer % 4 == 0 &&
        (reinterpret_cast<uintptr_t>(mask) & 3u) == 0 && n % 4 == 0) {
      // four consecutive elements (one row, contiguous flags) per thread:
      // one 16-byte LDS read and one 4-byte store; element 4j = q * inner_n + r
      const float4* c4 = reinterpret_cast<const float4*>(acache);
      const int64_t n4 = n / 4;
      int64_t q = 0, r = 4 * (int64_t)threadIdx.x;
      while (r >= pop.inner_n) {
        r -= pop.inner_n;
        ++q;
      }
      for (int64_t j = threadIdx.x; j < n4; j += NT) {
        const float4 a = c4[j];
        const uint32_t f = ((double)a.x > T ? 1u : 0u) | ((double)a.y > T ? 1u << 8 : 0u) |
                           ((double)a.z > T ? 1u << 16 : 0u) | ((double)a.w > T ? 1u << 24 : 0u);
        *reinterpret_cast<uint32_t*>(mask + pop.base + q * pop.s_outer + r) = f;
        r += 4 * NT;
        while (r >= pop.inner_n) {
          r -= pop.inner_n;
          ++q;
        }
      }
    } else if (cached && pop.inner_n >= NT) {
      // element i = q * inner_n + r; a step of NT carries into q at most once
      int64_t q = 0, r = threadIdx.x;
      for (int64_t i = threadIdx.x; i < n; i += NT) {
        mask[pop.base + q * pop.s_outer + r * pop.s_inner] = (double)amp(i) > T ? 1 : 0;
        r += NT;
        if (r >= pop.inner_n) {
          r -= pop.inner_n;
          ++q;
        }
      }
    } else {
      for_keys<NT, float>(n, amp, [&](int64_t i, float a) { mask[pop.off(i)] = (double)a > T ? 1 : 0; });
    }
  }
  if (threadIdx.x == 0) {
    if (thresh) thresh[id] = T;
    if (stats) {
      stats[2 * id] = med;
      stats[2 * id + 1] = madv;
    }
  }
}

#pragma clang fp contract(on)

constexpr int64_t MAD_CAP_BIG = 36864;   // floats cached in LDS (144 KiB)
constexpr int64_t MAD_CAP_SMALL = 2048;
constexpr int64_t MAD_LDS_FLOATS = 38400;  // dynamic LDS of the 1024-thread kernel: cache + compaction
constexpr int64_t MAD_COMP_MAX = 32768;

// The one-pass route takes populations of contiguous rows (all but the
// per-channel ones) that do not fit the LDS of one workgroup.  Below, mad_kernel
// alone takes 44 us for ten populations of 32768 with their amplitude pass
// (its selection passes read LDS), the three steps and the check 59 us.  Of
// populations no more than the compute units, whose time is that of one
// workgroup without the route, they have to be somewhat larger, the more so
// where elements are read one by one (vec false): one to 66 populations of
// 37000 take 61 to 74 us without and 64 to 76 with it (77 to 92 one by one), of
// 48000 74 to 84 and 65 to 77 (80 to 98), of 64000 85 to 101 and 68 to 80 (82 to
// 102).
bool mad_scans(int64_t npop, int64_t count, int population, bool vec) {
  const int64_t least = npop > device_cu_count() ? MAD_CAP_BIG + 1 : vec ? 42000 : 60000;
  return population != 1 && count >= least && count <= 0x7fffffffLL &&
         npop * ((count + MAD_CHUNK - 1) / MAD_CHUNK) <= 0x7fffffffLL;
}

int64_t mad_scratch_floats(int64_t n_time, int64_t n_base, int n_chan, int population) {
  const int64_t npop = population == 0 ? n_base : population == 1 ? n_base * n_chan : n_time * n_base;
  const int64_t count = population == 0 ? n_time * n_chan : population == 1 ? n_time : n_chan;
  if (population != 1 && count > MAD_CAP_BIG)
    return (npop * count + 1) / 2 * 2 + npop * (int64_t)(sizeof(MadWin) / sizeof(float));
  return count > MAD_CAP_SMALL ? npop * count : 0;
}

hipError_t launch_mad(const float2* vis, int64_t n_time, int64_t n_base, int n_chan, float sigma,
                      int population, uint8_t* mask, double* thresh, double* stats, float* amp_scratch,
                      hipStream_t s) {
  const int64_t npop = population == 0 ? n_base : population == 1 ? n_base * n_chan : n_time * n_base;
  const int64_t count = population == 0 ? n_time * n_chan : population == 1 ? n_time : n_chan;
  if (npop <= 0) return hipSuccess;
  if (count <= MAD_CAP_SMALL) {
    const size_t lds = (size_t)count * sizeof(float);
    return launch(mad_kernel<64, 8>, dim3((unsigned)npop), dim3(64), lds, s, vis, n_time, n_base, n_chan, sigma,
                  population, MAD_CAP_SMALL, (int64_t)0, nullptr, nullptr, mask, thresh, stats);
  } else {
    MadWin* win = nullptr;
    float* gamp = nullptr;
    const bool vec = n_chan % 4 == 0 && (reinterpret_cast<uintptr_t>(vis) & 15u) == 0 &&
                     (reinterpret_cast<uintptr_t>(mask) & 3u) == 0;
    if (amp_scratch && mad_scans(npop, count, population, vec)) {
      float* const lists = amp_scratch;
      win = reinterpret_cast<MadWin*>(amp_scratch + (npop * count + 1) / 2 * 2);
      const int chunks = (int)((count + MAD_CHUNK - 1) / MAD_CHUNK);
      hipError_t e = launch(vec ? mad_sample_kernel<true> : mad_sample_kernel<false>, dim3((unsigned)npop),
                            dim3(MAD_SAMPLE_NT), 0, s, vis, n_time, n_base, n_chan, sigma, population, win);
      if (e == hipSuccess)
        e = launch(vec ? mad_scan_kernel<true> : mad_scan_kernel<false>, dim3((unsigned)(npop * chunks)),
                   dim3(256), 0, s, vis, n_time, n_base, n_chan, population, chunks, win, lists, mask);
      if (e == hipSuccess)
        e = npop <= device_cu_count()
                ? launch(mad_finish_kernel<1024>, dim3((unsigned)npop), dim3(1024), 0, s, n_time, n_base, n_chan,
                         sigma, population, win, lists, mask, thresh, stats)
                : launch(mad_finish_kernel<512>, dim3((unsigned)npop), dim3(512), 0, s, n_time, n_base, n_chan, sigma,
                         population, win, lists, mask, thresh, stats);
      if (e != hipSuccess) return e;
      gamp = lists;
    }
    const int64_t cap = count <= MAD_CAP_BIG ? count : 0;
    if (amp_scratch && !win) {
      // the amplitudes are formed once, by the whole GPU: the selection
      // workgroups (one per population) then load 4 contiguous bytes per
      // element instead of forming a float64 square root each, and
      // populations beyond the LDS cache read 4 bytes per pass
      const int64_t total = npop * count;
      hipError_t e;
      if (population == 0 && n_chan % 4 == 0 && (reinterpret_cast<uintptr_t>(vis) & 31u) == 0 &&
          (reinterpret_cast<uintptr_t>(amp_scratch) & 15u) == 0) {
        const int64_t total4 = total / 4;
        e = launch(mad_amp4_kernel, dim3((unsigned)((total4 + 255) / 256)), dim3(256), 0, s,
                   reinterpret_cast<const float4*>(vis), n_base, n_chan, count, total4,
                   reinterpret_cast<float4*>(amp_scratch));
      } else {
        e = launch(mad_amp_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, vis, n_time, n_base,
                   n_chan, population, count, total, amp_scratch);
      }
      if (e != hipSuccess) return e;
      gamp = amp_scratch;
    }
    // what LDS the cache leaves holds the compaction buffer
    int64_t comp_cap = MAD_LDS_FLOATS - cap;
    comp_cap = comp_cap < MAD_COMP_MAX ? comp_cap : MAD_COMP_MAX;
    if (comp_cap < 256) comp_cap = 0;
    const size_t lds = (size_t)(cap + comp_cap) * sizeof(float);
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(mad_kernel<1024, 11>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    return launch(mad_kernel<1024, 11>, dim3((unsigned)npop), dim3(1024), lds, s, vis, n_time, n_base, n_chan,
                  sigma, population, cap, comp_cap, gamp, win, mask, thresh, stats);
  }
}

// ---------------------------------------------------------------------------
// Delay/phase application.
// ---------------------------------------------------------------------------
constexpr int APPLY_MAX_ANT = 64;
struct AntTable {
  double tau[APPLY_MAX_ANT];
  double phi[APPLY_MAX_ANT];
};

__global__ void __launch_bounds__(256)
apply_kernel(float2* __restrict__ vis, int n_ant, int n_chan, double f0, double df, AntTable t) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n_chan) return;
  int b = blockIdx.y, i = 0;
  while (b >= n_ant - i) { b -= n_ant - i; ++i; }
  const int j = i + b;
  if (i == j) return;  // zero rotation: autos unchanged
  const double inv2pi = 0.15915494309189533577;
  const double fk = f0 + (double)k * df;
  double cyc = fk * (t.tau[i] - t.tau[j]) + (t.phi[i] - t.phi[j]) * inv2pi;
  cyc -= rint(cyc);
  double sn, cs;
  sincospi(2.0 * cyc, &sn, &cs);
  const int64_t nb = (int64_t)n_ant * (n_ant + 1) / 2;
  float2* p = vis + ((int64_t)blockIdx.z * nb + blockIdx.y) * n_chan + k;
  const float2 v = *p;
  const double re = (double)v.x * cs - (double)v.y * sn;
  const double im = (double)v.x * sn + (double)v.y * cs;
  *p = make_float2((float)re, (float)im);
}

hipError_t launch_apply(float2* vis, int64_t n_time, int n_ant, int n_chan, double f0, double df,
                        const double* tau, const double* phi, hipStream_t s) {
  if (n_ant > APPLY_MAX_ANT) return hipErrorInvalidValue;
  AntTable t{};
  for (int a = 0; a < n_ant; ++a) {
    t.tau[a] = tau[a];
    t.phi[a] = phi[a];
  }
  const int nb = n_ant * (n_ant + 1) / 2;
  if (n_time <= 0 || nb <= 0 || n_chan <= 0) return hipSuccess;
  dim3 grid((unsigned)((n_chan + 255) / 256), (unsigned)nb, (unsigned)n_time);
  return launch(apply_kernel, grid, dim3(256), 0, s, vis, n_ant, n_chan, f0, df, t);
}

}  // namespace qc
