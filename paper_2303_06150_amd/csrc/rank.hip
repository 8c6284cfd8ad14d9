// Global ranking of a library (Sec. 2: rank the input chemical library by the
// docked ligands' scores): the top m of n groups by each group's best value,
// equal values ordered by lower group index.
//
// Keys.  Group i with best value v has a 64-bit key: the upper word orders the
// values (larger value, larger key; -0 counts as +0), the lower word is
// 0xFFFFFFFF - i, so equal values rank the lower index first.  Keys are
// distinct, so "the top m" is a set and no sort stability is needed.  Only the
// upper words are stored; the lower ones follow from the position.
//
// Steps.  (1) upper words, with the histogram of their top 11 bits; (2) radix
// select of the m-th largest key by six digits of 11, 11, 10 bits of each word:
// every pass first picks the digit's bin from the histogram of the pass before
// (each block for itself), then counts the next digit of the keys that match,
// and does nothing once few enough keys are left to finish by comparison;
// (3) compaction of the keys at or above the last threshold; (4) m <= 4096: the
// place of each of the at most 4096 candidates is the number of larger ones,
// counted in LDS, and the result goes straight to its place; larger m: a
// descending bitonic sort of the m keys (tile sorts in LDS, global merge steps).
//
// What bounds it: the launches (nine of 2 to 6 us), then the read of the scores.
// One million groups of eight values, m = 1000, a whole call: 156 us with byte
// digits (a histogram and a pick launch each, 64-bit keys read up to nine times)
// and a sort of the candidates by one block, 59 us with the keys' values staged
// through LDS (29 us for 32 MB), 41 us as it is.
// At most 4096 groups: one launch or two.
#include "lg.h"
#include "lg_internal.h"

#include <algorithm>
#include <mutex>

namespace lg {

namespace {

constexpr int kTile = 4096;          // keys sorted in LDS by one block (32 KB)
constexpr int kSortThreads = 1024;

__device__ __forceinline__ uint64_t rank_key(float v, int i) {
  const uint32_t hi = (uint32_t)orderable(v + 0.0f) ^ 0x80000000u;
  return ((uint64_t)hi << 32) | (uint64_t)(0xFFFFFFFFu - (uint32_t)i);
}

__device__ __forceinline__ float key_value(uint64_t k) {
  const int o = (int)((uint32_t)(k >> 32) ^ 0x80000000u);
  return __int_as_float(o ^ ((o >> 31) & 0x7FFFFFFF));   // orderable() is its own inverse
}

__device__ __forceinline__ int key_index(uint64_t k) { return (int)(0xFFFFFFFFu - (uint32_t)k); }

// Best value of a group and the first member that has it.
__device__ __forceinline__ float group_best(const float* s, int group, int* member) {
  float best = s[0];
  int bm = 0;
  for (int q = 1; q < group; ++q)
    if (s[q] > best) { best = s[q]; bm = q; }
  *member = bm;
  return best;
}

// Best value of a group by a row of 16 lanes, on every lane of it: the first value's if
// that is NaN, else the largest of those that are not (as group_best has it).
__device__ __forceinline__ float row_best(const float* s, int group) {
  float best = s[0];
  if (best != best) return best;
#pragma unroll 4
  for (int q = threadIdx.x & 15; q < group; q += 16) best = s[q] > best ? s[q] : best;
#pragma unroll
  for (int o = 1; o < 16; o *= 2) {
    const float other = __shfl_xor(best, o);
    best = other > best ? other : best;
  }
  return best;
}

// Value words of long groups, a row of 16 lanes each.
__global__ __launch_bounds__(256) void rank_words_kernel(const float* score, int n, int group, uint32_t* words) {
  const int g = blockIdx.x * 16 + ((int)threadIdx.x >> 4);
  if (g >= n) return;
  const uint32_t w = (uint32_t)(rank_key(row_best(score + (long long)g * group, group), 0) >> 32);
  if ((threadIdx.x & 15) == 0) words[g] = w;
}

// Digits of the 64-bit key from the top: 11, 11, 10 bits of the value word, then
// of the index word.
// The digits' histograms take three places in turn: one is read, one filled and one
// cleared for the next pass.
constexpr int kDigits = 6, kBins = 2048, kHists = 3;
__device__ __forceinline__ int digit_shift(int d) { return d == 0 ? 53 : d == 1 ? 42 : d == 2 ? 32 : d == 3 ? 21 : d == 4 ? 10 : 0; }
__device__ __forceinline__ uint32_t digit_mask(int d) { return d % 3 == 2 ? 1023u : 2047u; }

__global__ void rank_init_kernel(RankState* st, uint32_t* hist, int m) {
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    st[0].prefix = 0;
    st[0].mask = 0;
    st[0].need = (uint32_t)m;
    st[0].done = 0;
    st[0].count = 0;
    st[kDigits].count = 0;   // candidates
  }
  // the first two digits'; every later one is cleared by the pass before it
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < 2 * kBins; i += gridDim.x * blockDim.x) hist[i] = 0;
}

__device__ __forceinline__ void add_bins(const uint32_t* lh, uint32_t* hist) {
  __syncthreads();
  for (int b = threadIdx.x; b < kBins; b += blockDim.x)
    if (lh[b]) atomicAdd(&hist[b], lh[b]);
}

// Value words of all groups and the histogram of their top digit.  Bound by the
// read of the scores, so by the bytes in flight.  VEC (groups of whole, aligned
// float4): a thread reads its groups' values itself, kGroupsInFlight groups at a
// time; few large blocks, because each adds its histogram to the global one and
// those additions are contended (a whole ranking of one million groups of eight:
// 59 us through LDS, 43 with 512 blocks of 256, 41 with 256 of 1 024).  Otherwise a
// block takes 256 groups at a time, whose values are one stretch, read coalesced
// into LDS (groups of up to kStageGroup values); longer ones, and any from kLongGroup
// values on, are read by rows of 16 lanes, 16 groups a block and time (50 000 groups of
// 200: a thread a group leaves 25 blocks of work, 168 us a call; 92 so).
constexpr int kStageGroup = 24, kLongGroup = 64;
constexpr int kGroupsInFlight = 2, kKeyThreads = 1024;

template <bool VEC>
__global__ __launch_bounds__(VEC ? kKeyThreads : 256) void rank_keys_kernel(const float* score, int n, int group,
                                                                            uint32_t* words, uint32_t* hist) {
  __shared__ uint32_t lh[kBins];
  for (int b = threadIdx.x; b < kBins; b += blockDim.x) lh[b] = 0;
  __syncthreads();
  auto put = [&](long long g, float v) {
    const uint32_t w = (uint32_t)(rank_key(v, 0) >> 32);
    words[g] = w;
    atomicAdd(&lh[w >> 21], 1u);
  };
  if constexpr (VEC) {
    constexpr int U = kGroupsInFlight;
    for (long long g0 = blockIdx.x * ((long long)kKeyThreads * U); g0 < n; g0 += gridDim.x * ((long long)kKeyThreads * U)) {
      const float4* src[U];
      float best[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {   // past the last group: that one again, not stored
        const long long g = min(g0 + kKeyThreads * u + threadIdx.x, n - 1LL);
        src[u] = reinterpret_cast<const float4*>(score + g * group);
      }
      auto add = [&](float v, float& b) { b = v > b ? v : b; };
      for (int t = 0; t < group / 4; t += 2) {
        const int t1 = min(t + 1, group / 4 - 1);   // an odd count: the last four again, which changes nothing
        float4 q[U], r[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          q[u] = src[u][t];
          r[u] = src[u][t1];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if (t == 0) best[u] = q[u].x;
          add(q[u].x, best[u]);
          add(q[u].y, best[u]);
          add(q[u].z, best[u]);
          add(q[u].w, best[u]);
          add(r[u].x, best[u]);
          add(r[u].y, best[u]);
          add(r[u].z, best[u]);
          add(r[u].w, best[u]);
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const long long g = g0 + kKeyThreads * u + threadIdx.x;
        if (g < n) put(g, best[u]);
      }
    }
  } else {
    __shared__ float vals[256 * kStageGroup];
    if (group > kStageGroup) {
      for (long long g = blockIdx.x * 16LL + (threadIdx.x >> 4); g < n; g += gridDim.x * 16LL) {
        const float best = row_best(score + g * group, group);
        if ((threadIdx.x & 15) == 0) put(g, best);
      }
    } else {
      for (long long g0 = blockIdx.x * 256LL; g0 < n; g0 += gridDim.x * 256LL) {
        const int groups = (int)min(256LL, n - g0);
        const float* src = score + g0 * group;
        for (int t = threadIdx.x; t < groups * group; t += 256) vals[t] = src[t];
        __syncthreads();
        if ((int)threadIdx.x < groups) {
          int member;
          put(g0 + threadIdx.x, group_best(vals + (int)threadIdx.x * group, group, &member));
        }
        __syncthreads();
      }
    }
  }
  add_bins(lh, hist);
}

// Digit d's bin of the key of rank `need` (counting from the largest) among the
// keys matching the state's prefix, by all 256 threads of a block: the state
// with the prefix extended by it.  Done once the keys at or above the extended
// prefix are at most `room` (m for an exact selection): then those are the
// candidates.
__device__ __forceinline__ RankState rank_pick(RankState st, const uint32_t* hist, int d, uint32_t room, uint32_t m) {
  __shared__ uint32_t above_s[257];
  __shared__ RankState out;
  if (st.done) return st;
  constexpr int PER = kBins / 256;
  // bins from the top: thread t has bins kBins - 1 - PER t downwards
  uint32_t mine[PER], sum = 0;
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    mine[k] = hist[kBins - 1 - PER * (int)threadIdx.x - k];
    sum += mine[k];
  }
  // exclusive prefix of the sums over the block
  const int lane = lane_id(), wave = threadIdx.x >> 6;
  uint32_t incl = sum;
#pragma unroll
  for (int o = 1; o < 64; o *= 2) {
    const uint32_t v = __shfl_up(incl, o);
    if (lane >= o) incl += v;
  }
  if (lane == 63) above_s[wave] = incl;
  __syncthreads();
  uint32_t above = incl - sum;
  for (int w = 0; w < wave; ++w) above += above_s[w];
  if (above < st.need && above + sum >= st.need) {   // exactly one thread
    int k = 0;
#pragma unroll
    for (; k < PER - 1; ++k) {
      if (above + mine[k] >= st.need) break;
      above += mine[k];
    }
    const uint32_t bin = (uint32_t)(kBins - 1 - PER * (int)threadIdx.x - k);
    uint32_t held = 0;
#pragma unroll
    for (int q = 0; q < PER; ++q) held = q == k ? mine[q] : held;
    RankState r = st;
    r.need = st.need - above;
    r.prefix |= (uint64_t)bin << digit_shift(d);
    r.mask |= (uint64_t)digit_mask(d) << digit_shift(d);
    r.done = m - r.need + held <= room ? 1u : 0u;   // larger keys, and those of this bin
    r.count = 0;
    out = r;
  }
  __syncthreads();
  return out;
}

// Keys i0 .. i1 - 1 (i0 a multiple of 4) handed to f, four words a read and two
// reads in flight, by thread `t` of `threads`.  The words' space is whole float4.
template <class F>
__device__ __forceinline__ void for_each_key(const uint32_t* words, long long i0, long long i1, int t, int threads, F f) {
  const uint4* q = reinterpret_cast<const uint4*>(words);
  const long long end = (i1 + 3) / 4;
  for (long long j = i0 / 4 + t; j < end; j += 2LL * threads) {
    const long long j2 = j + threads;
    const uint4 a = q[j], b = q[min(j2, end - 1)];
    const uint32_t w[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const long long i = 4 * (e < 4 ? j : j2) + (e & 3);
      if (i < i1) f(((uint64_t)w[e] << 32) | (uint64_t)(0xFFFFFFFFu - (uint32_t)i));
    }
  }
}

// Digit d - 1 picked, digit d counted among the keys that match it.
__global__ __launch_bounds__(256) void rank_digit_kernel(const uint32_t* words, int n, RankState* states,
                                                         uint32_t* hist, int d, uint32_t room, uint32_t m) {
  __shared__ uint32_t lh[kBins];
  const RankState st = rank_pick(states[d - 1], hist + (d - 1) % kHists * kBins, d - 1, room, m);
  if (blockIdx.x == 0 && threadIdx.x == 0) states[d] = st;
  if (st.done) return;
  for (int b = blockIdx.x * 256 + threadIdx.x; b < kBins; b += gridDim.x * 256) hist[(d + 1) % kHists * kBins + b] = 0;
  for (int b = threadIdx.x; b < kBins; b += blockDim.x) lh[b] = 0;
  __syncthreads();
  const int shift = digit_shift(d);
  const uint32_t bins = digit_mask(d);
  for_each_key(words, 0, n, blockIdx.x * 256 + threadIdx.x, gridDim.x * 256, [&](uint64_t k) {
    if ((k & st.mask) == st.prefix) atomicAdd(&lh[(uint32_t)(k >> shift) & bins], 1u);
  });
  add_bins(lh, hist + d % kHists * kBins);
}

// The keys at or above the threshold (at most `room`), in any order, and their
// number; `fill` keys after them set to 0 (for the bitonic sort).  Each block
// counts the keys of its stretch, takes their places with one addition to the
// global counter (a contended addition costs about 30 ns) and reads them again.
__global__ __launch_bounds__(256) void rank_compact_kernel(const uint32_t* words, int n, RankState* states,
                                                           const uint32_t* hist, uint64_t* cand, uint32_t room,
                                                           uint32_t m, long long fill) {
  __shared__ uint32_t taken, base;
  const RankState st = rank_pick(states[kDigits - 1], hist + (kDigits - 1) % kHists * kBins, kDigits - 1, room, m);
  const uint64_t t = st.prefix;
  const long long per = ((n + (long long)gridDim.x - 1) / gridDim.x + 255) / 256 * 256;
  const long long i0 = blockIdx.x * per, i1 = min((long long)n, i0 + per);
  if (threadIdx.x == 0) taken = 0;
  __syncthreads();
  uint32_t mine = 0;
  for_each_key(words, i0, i1, threadIdx.x, 256, [&](uint64_t k) { mine += k >= t ? 1u : 0u; });
  mine = (uint32_t)wave_reduce_i32((int)mine, OpAdd());
  if (lane_id() == 0 && mine) atomicAdd(&taken, mine);
  __syncthreads();
  if (threadIdx.x == 0) {
    base = taken ? atomicAdd(&states[kDigits].count, taken) : 0;   // zeroed with the histograms
    taken = 0;
  }
  __syncthreads();
  for_each_key(words, i0, i1, threadIdx.x, 256, [&](uint64_t k) {
    if (k < t) return;
    const uint32_t at = base + atomicAdd(&taken, 1u);
    if (at < room) cand[at] = k;
  });
  for (long long i = m + blockIdx.x * 256LL + threadIdx.x; i < fill; i += gridDim.x * 256LL) cand[i] = 0;
}

// Result q: group, value and member of key k.
__device__ __forceinline__ void rank_store(uint64_t k, int q, const float* score, int n, int group, int32_t* top_idx,
                                           float* top_score, int32_t* top_member) {
  const int i = key_index(k);
  top_idx[q] = i;
  top_score[q] = key_value(k);
  if (top_member) {
    int member = -1;
    if (i >= 0 && i < n) group_best(score + (long long)i * group, group, &member);
    top_member[q] = member;
  }
}

// Places of the `count` keys in LDS by counting the larger ones: the block places
// kPlaces of them, 16 threads to a key, and stores those of the top m.
constexpr int kPlaces = 16;

__device__ __forceinline__ void rank_place(const uint64_t* s, int count, const float* score, int n, int group, int m,
                                           int32_t* top_idx, float* top_score, int32_t* top_member) {
  const int c = blockIdx.x * kPlaces + ((int)threadIdx.x >> 4), part = threadIdx.x & 15;
  const uint64_t k = c < count ? s[c] : 0;
  int larger = 0;
#pragma unroll 4
  for (int t = part; t < count; t += 16) larger += s[t] > k ? 1 : 0;
#pragma unroll
  for (int o = 1; o < 16; o *= 2) larger += __shfl_xor(larger, o);
  if (part == 0 && c < count && larger < m) rank_store(k, larger, score, n, group, top_idx, top_score, top_member);
}

// At most kTile candidates.
__global__ __launch_bounds__(256) void rank_place_kernel(const uint64_t* cand, const RankState* states,
                                                         const float* score, int n, int group, int m,
                                                         int32_t* top_idx, float* top_score, int32_t* top_member) {
  __shared__ uint64_t s[kTile];
  const int count = min((int)states[kDigits].count, kTile);
  if ((int)blockIdx.x * kPlaces >= count) return;
  for (int t = threadIdx.x; t < count; t += 256) s[t] = cand[t];
  __syncthreads();
  rank_place(s, count, score, n, group, m, top_idx, top_score, top_member);
}

// The ranking of at most kTile groups: every block takes all keys and places kPlaces.
// Without stored words it takes them from the scores, one launch for everything, up to
// kSmallValues values: each block reads them all, out of the L2 (4 096 groups: 44 us for
// groups of 8, 74 of 24, 117 of 32, 200 of 64; the same 64 k values in 1 000 groups 61 us).
// More values are read once, into words, by a launch before it.
constexpr long long kSmallValues = 1 << 16;

__global__ __launch_bounds__(256) void rank_small_kernel(const uint32_t* words, const float* score, int n, int group, int m,
                                                         int32_t* top_idx, float* top_score, int32_t* top_member) {
  __shared__ uint64_t s[kTile];
  for (int t = threadIdx.x; t < n; t += 256) {
    int member;
    s[t] = words ? (uint64_t)words[t] << 32 | (uint64_t)(0xFFFFFFFFu - (uint32_t)t)
                 : rank_key(group_best(score + (long long)t * group, group, &member), t);
  }
  __syncthreads();
  rank_place(s, n, score, n, group, m, top_idx, top_score, top_member);
}

// One compare-exchange of the descending bitonic network: stage k, distance j.
__device__ __forceinline__ void bitonic_cx(uint64_t& a, uint64_t& b, long long i, long long k) {
  const bool desc = (i & k) == 0;
  if (desc ? a < b : a > b) {
    const uint64_t t = a;
    a = b;
    b = t;
  }
}

// Sort of `len` (power of two, <= kTile) keys in LDS, stages k0 (first) to
// kmax, then writes them back.  With k0 = 2 a whole tile is sorted; with
// k0 = kmax > kTile only the steps j < kTile of stage kmax run (the merge tail).
__global__ __launch_bounds__(kSortThreads) void rank_tile_kernel(uint64_t* a, int len, long long k0, long long kmax) {
  __shared__ uint64_t s[kTile];
  const long long base = (long long)blockIdx.x * len;
  for (int t = threadIdx.x; t < len; t += blockDim.x) s[t] = a[base + t];
  __syncthreads();
  for (long long k = k0; k <= kmax; k *= 2) {
    for (long long j = (k > len ? len : k) / 2; j >= 1; j /= 2) {
      for (int p = threadIdx.x; p < len / 2; p += blockDim.x) {
        const int i = (int)(2 * j * (p / j) + (p % j));
        bitonic_cx(s[i], s[i + j], base + i, k);
      }
      __syncthreads();
    }
  }
  for (int t = threadIdx.x; t < len; t += blockDim.x) a[base + t] = s[t];
}

// One global step (stage k, distance j >= kTile) of the bitonic network.
__global__ __launch_bounds__(256) void rank_merge_kernel(uint64_t* a, long long padded, long long k, long long j) {
  const long long stride = (long long)gridDim.x * blockDim.x;
  for (long long p = blockIdx.x * (long long)blockDim.x + threadIdx.x; p < padded / 2; p += stride) {
    const long long i = 2 * j * (p / j) + (p % j);
    bitonic_cx(a[i], a[i + j], i, k);
  }
}

__global__ void rank_out_kernel(const uint64_t* sorted, const float* score, int n, int group, int m,
                                int32_t* top_idx, float* top_score, int32_t* top_member) {
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q < m) rank_store(sorted[q], q, score, n, group, top_idx, top_score, top_member);
}

long long pow2_at_least(long long m) {
  long long p = 1;
  while (p < m) p *= 2;
  return p;
}

constexpr size_t up256(size_t b) { return (b + 255) & ~(size_t)255; }

// Candidates of a ranking of the top m: up to kTile a quarter more than wanted will do
// (placing them costs less than another digit); more: exactly the top m, in the power
// of two of places that the bitonic sort needs.
constexpr uint32_t candidates(uint32_t m) {
  if (m > (uint32_t)kTile) return m;
  const uint32_t room = m + (m / 4 > 256 ? m / 4 : 256);
  return room < (uint32_t)kTile ? room : (uint32_t)kTile;
}

// Scratch of the selection: states, three histograms, value words, candidates.
constexpr size_t scratch_bytes(size_t n, size_t places) {
  return up256((kDigits + 1) * sizeof(RankState)) + up256(kHists * kBins * sizeof(uint32_t)) + up256(n * 4) +
         up256(places * 8);
}

// Fixed device scratch of lg_rank_static, sized for its largest accepted call
// (LG_RANK_STATIC_MAX_TOP is a power of two).  Every device the library runs on
// holds one copy until the process ends.  Host code must not pass this name to
// a kernel: its device address comes from hipGetSymbolAddress.
static_assert((LG_RANK_STATIC_MAX_TOP & (LG_RANK_STATIC_MAX_TOP - 1)) == 0, "power of two");
constexpr size_t kStaticScratchBytes = scratch_bytes(LG_RANK_STATIC_MAX_GROUPS, LG_RANK_STATIC_MAX_TOP > kTile ? LG_RANK_STATIC_MAX_TOP : kTile);
__device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

constexpr int kMaxDevices = 64;

}  // namespace

// Scratch of a call; never more than 12 bytes a group and 8 for every place of the power
// of two above m, plus the fixed part of 1 280 bytes, which an earlier selection took.
size_t rank_scratch_bytes(int n, int group, int m) {
  if (n <= kTile) return (long long)n * group <= kSmallValues ? 0 : up256((size_t)n * 4);
  return scratch_bytes((size_t)n, m > kTile ? (size_t)pow2_at_least(m) : candidates((uint32_t)std::max(m, 1)));
}

// Device address of the current device's copy of the fixed scratch, looked up
// once per device (with that device current) and kept.
hipError_t rank_static_scratch(void** out, size_t* bytes) {
  static std::mutex mu;
  static void* ptr[kMaxDevices] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> g(mu);
  if (!ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    ptr[dev] = p;
  }
  *out = ptr[dev];
  *bytes = kStaticScratchBytes;
  return hipSuccess;
}

hipError_t launch_rank(const float* score, int n, int group, int m, void* work, int32_t* top_idx,
                       float* top_score, int32_t* top_member, hipStream_t st) {
  if (n <= 0 || m <= 0) return hipSuccess;
  if (n <= kTile) {
    uint32_t* words = (long long)n * group <= kSmallValues ? nullptr : (uint32_t*)work;
    if (words) hipLaunchKernelGGL(rank_words_kernel, dim3((n + 15) / 16), dim3(256), 0, st, score, n, group, words);
    hipLaunchKernelGGL(rank_small_kernel, dim3((n + kPlaces - 1) / kPlaces), dim3(256), 0, st, words, score, n, group, m,
                       top_idx, top_score, top_member);
    return hipGetLastError();
  }
  char* w = (char*)work;
  RankState* states = (RankState*)w;
  w += up256((kDigits + 1) * sizeof(RankState));
  uint32_t* hist = (uint32_t*)w;
  w += up256(kHists * kBins * sizeof(uint32_t));
  uint32_t* words = (uint32_t*)w;
  w += up256((size_t)n * 4);
  uint64_t* cand = (uint64_t*)w;
  const long long padded = pow2_at_least(m);
  const bool one_tile = m <= kTile;
  const uint32_t room = candidates((uint32_t)m);
  // each block adds its histogram to the global one: at most one per compute unit (two
  // where the keys come through LDS or by rows), at least four groups per thread or row
  const auto share = [](long long count, long long per, long long most) {
    return (int)std::max<long long>(1, std::min<long long>((count + per - 1) / per, most));
  };
  const int few = share(n, 1024, 256);
  hipLaunchKernelGGL(rank_init_kernel, dim3(12), dim3(256), 0, st, states, hist, m);
  if (group % 4 == 0 && group < kLongGroup && (uintptr_t)score % 16 == 0)
    hipLaunchKernelGGL(rank_keys_kernel<true>, dim3(share(n, kKeyThreads * kGroupsInFlight, 256)), dim3(kKeyThreads), 0, st,
                       score, n, group, words, hist);
  else
    hipLaunchKernelGGL(rank_keys_kernel<false>, dim3(share(n, group > kStageGroup ? 64 : 1024, 512)), dim3(256), 0, st,
                       score, n, group, words, hist);
  for (int d = 1; d < kDigits; ++d)
    hipLaunchKernelGGL(rank_digit_kernel, dim3(few), dim3(256), 0, st, words, n, states, hist, d, room, (uint32_t)m);
  hipLaunchKernelGGL(rank_compact_kernel, dim3(few), dim3(256), 0, st, words, n, states, hist, cand, room,
                     (uint32_t)m, one_tile ? 0LL : padded);
  if (one_tile) {
    hipLaunchKernelGGL(rank_place_kernel, dim3((room + kPlaces - 1) / kPlaces), dim3(256), 0, st, cand, states, score, n, group, m, top_idx,
                       top_score, top_member);
    return hipGetLastError();
  }
  const int tiles = (int)(padded / kTile);
  const int mblocks = (int)std::min<long long>(padded / 2 / 256, 4096);
  hipLaunchKernelGGL(rank_tile_kernel, dim3(tiles), dim3(kSortThreads), 0, st, cand, kTile, 2LL, (long long)kTile);
  for (long long k = 2LL * kTile; k <= padded; k *= 2) {
    for (long long j = k / 2; j >= kTile; j /= 2)
      hipLaunchKernelGGL(rank_merge_kernel, dim3(mblocks), dim3(256), 0, st, cand, padded, k, j);
    hipLaunchKernelGGL(rank_tile_kernel, dim3(tiles), dim3(kSortThreads), 0, st, cand, kTile, k, k);
  }
  hipLaunchKernelGGL(rank_out_kernel, dim3((m + 255) / 256), dim3(256), 0, st, cand, score, n, group, m, top_idx,
                     top_score, top_member);
  return hipGetLastError();
}

}  // namespace lg
