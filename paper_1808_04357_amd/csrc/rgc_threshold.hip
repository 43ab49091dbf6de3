// gfx950 kernels of the compression step with threshold binary search selection (RedSync,
// Section 2.1, Algorithm 3, and the sampled variant of the same section that reuses a threshold):
// the communication-set of a layer is every element whose magnitude exceeds a threshold, the
// threshold is searched on  mean + ratio * (max - mean),  ratio bisected in [0, 1] until between
// k and 2k elements pass or the interval is shorter than 2^-10.
//
// The paper's listing counts the elements above the threshold once per bisection step, i.e. up to
// ten passes over the layer.  Here the ten counts cost ONE pass: the interval ends are multiples
// of 2^-10, so the search can only ever try the 1023 thresholds  T(j) = mean + (j/1024)(max - mean);
// a histogram of  bin(x) = #{j : T(j) < |x|}  over the layer gives the count above every T(j) as a
// suffix sum, and the bisection runs on those sums.  T(j) is computed with the very operations
// of the listing (fp32, every operation rounded), so the counts are the listing's counts.
//
// And that pass goes over lists of the layer's largest elements, not over the layer.  A sample of the accumulated values
// (16384 of them, from 1024 places) gives a magnitude that about 4k elements exceed; the streaming pass
// lists those.  If it has listed at least 2k of them, every count the search compares with k and 2k is known: above a
// threshold not below that magnitude from the lists, above a lower one it is 2k or more, and that is all the search asks.
// LSTM set: 291 us per call with three more passes over V, 212 us this way.
// A layer whose lists do not do (too few listed, a list that ran over, a share too large to list, a search that ends below)
// is read from V instead, in the same launches.
//
// Launches of one call (same workgroup -> layer -> wave-chunk decomposition as the exact path):
//   search:  sample  ->  accumulate (+ partial sums and maxima of |a|, lists)  ->  moments  ->  histogram  ->  search
//            ->  count  ->  emit
//   reuse:   accumulate (+ the elements above the given threshold, listed per wave-chunk)
//            ->  emit from the lists
//   and a launch that scans the counts of very large layers before emit
#include "rgc_exact.h"

namespace rgc {

namespace {

constexpr uint32_t kSteps = 1024;   // 1 / epsilon of the search: ratios are multiples of 2^-10
constexpr uint32_t kHistReps = static_cast<uint32_t>(kHistBins) / kSteps;   // copies of a histogram of that many bins

typedef uint32_t vu2 __attribute__((ext_vector_type(2)));   // a listed element: (float bits, index)

// T(j), j = 1 .. 1023; the operations and their order are those of Algorithm 3.
__device__ __forceinline__ float threshold_at(float mean, float span, uint32_t j) {
  const float ratio = static_cast<float>(j) * (1.0f / static_cast<float>(kSteps));   // exact
  return __fadd_rn(mean, __fmul_rn(ratio, span));
}

// #{j in 1..1023 : T(j) < x}.  T is non-decreasing in j (span >= 0, rounding is monotone), so this is
// the largest j with T(j) < x, or 0.  A guess from the inverse map is checked against T itself; where
// the guess is off, a binary search over j finds it.
__device__ __forceinline__ uint32_t bin_of(float x, float mean, float span, float inv) {
  const float g = __fmul_rn(__fsub_rn(x, mean), inv);
  uint32_t j = g > 0.0f ? (g < static_cast<float>(kSteps - 1u) ? static_cast<uint32_t>(g) : kSteps - 1u) : 0u;   // NaN -> 0
  const bool lo_ok = (j == 0u) || (threshold_at(mean, span, j) < x);
  const bool hi_ok = (j == kSteps - 1u) || !(threshold_at(mean, span, j + 1u) < x);
  if (lo_ok && hi_ok) return j;
  uint32_t lo = 0u, hi = kSteps - 1u;
  while (lo < hi) {
    const uint32_t mid = (lo + hi + 1u) >> 1;
    if (threshold_at(mean, span, mid) < x) lo = mid; else hi = mid - 1u;
  }
  return lo;
}

struct Place {           // where a wave works
  uint32_t l;            // layer
  uint32_t wc;           // its wave-chunk, global number
  uint32_t begin, end;   // element range inside the layer; begin == end: nothing to do
};

__device__ __forceinline__ Place place_of(const ThresholdArgs& A, const LayerDesc& L, uint32_t l, uint32_t wg) {
  Place p;
  p.l = l;
  const uint32_t wc_local = (wg - L.wg_first) * kWavesPerBlock + (threadIdx.x >> 6);
  p.wc = L.wc_first + wc_local;
  if (wc_local < L.wc_count) {
    p.begin = wc_local * A.chunk;
    p.end = (L.n - p.begin) < A.chunk ? L.n : p.begin + A.chunk;
  } else {
    p.begin = p.end = 0u;
  }
  return p;
}

// Calls f(a, nvalid, idx0) for the groups of 256 elements of [begin, end) of tensor p: lane-major,
// four consecutive elements per lane; whole groups four at a time.
template <typename F>
__device__ __forceinline__ void read_groups(const float* generic_p, uint32_t begin, uint32_t end, F&& f) {
  const gptr<const float> p = as_global(generic_p);
  const uint32_t lane = lane_id();
  uint32_t base = begin;
  {
    constexpr uint32_t kUnroll = 4u;
    for (; base + kUnroll * kGroupElems <= end; base += kUnroll * kGroupElems) {
      vf4 q[kUnroll];
#pragma unroll
      for (uint32_t t = 0; t < kUnroll; ++t) q[t] = *as_vec(generic_p + base + t * kGroupElems + lane * 4u);
#pragma unroll
      for (uint32_t t = 0; t < kUnroll; ++t) {
        const float a[4] = {q[t].x, q[t].y, q[t].z, q[t].w};
        f(a, 4u, base + t * kGroupElems + lane * 4u);
      }
    }
  }
  for (; base < end; base += kGroupElems) {
    const uint32_t idx0 = base + lane * 4u;
    float a[4] = {0.f, 0.f, 0.f, 0.f};
    uint32_t nvalid;
    if (base + kGroupElems <= end) {
      const vf4 q = *as_vec(generic_p + idx0);
      a[0] = q.x; a[1] = q.y; a[2] = q.z; a[3] = q.w;
      nvalid = 4u;
    } else {
      nvalid = idx0 < end ? ((end - idx0) < 4u ? (end - idx0) : 4u) : 0u;
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (static_cast<uint32_t>(j) < nvalid) a[j] = p[idx0 + j];
    }
    f(a, nvalid, idx0);
  }
}

// Calls f(entry, exists) for the entries of the wave-chunk's list, 64 at a time (all lanes take part).
template <typename F>
__device__ __forceinline__ void for_listed(const ThresholdArgs& A, const Place& p, F&& f) {
  if (p.begin == p.end) return;
  const gptr<const vu2> slot = as_global(reinterpret_cast<const vu2*>(A.slots + static_cast<size_t>(p.wc) * A.cap));
  const uint32_t lane = lane_id();
  vu2 e = slot[lane];                               // (the slots exist whatever the length: a list has more than 64)
  const uint32_t listed = A.listed[p.wc] < A.cap ? A.listed[p.wc] : A.cap;
  for (uint32_t b = 0; b < listed; b += kWaveSize) {
    const vu2 next = b + kWaveSize + lane < listed ? slot[b + kWaveSize + lane] : vu2{0u, 0u};
    f(e, b + lane < listed);
    e = next;
  }
}

// The accumulate of Algorithm 1 over [begin, end) of a layer (same arithmetic as the exact path:
// accum4), handing every group of accumulated values to f.
template <bool kNt, bool kMom, bool kNest, typename F>
__device__ __forceinline__ void accumulate_groups(const LayerDesc& L, uint32_t begin, uint32_t end, const AccumRule& rule, F&& f) {
  const gptr<const float> G = as_global(L.grad);
  const gptr<float> V = as_global(L.resid);
  const gptr<float> U = as_global(L.mom);
  const uint32_t lane = lane_id();
  uint32_t base = begin;
  {
    const uint32_t groups = __builtin_amdgcn_readfirstlane((end - begin) / kGroupElems);
    const gvf4 V4 = as_vec(L.resid + begin);
    const gvf4 U4 = kMom ? as_vec(L.mom + begin) : nullptr;
    stream_groups<kNt, kMom, 4>(as_vec(L.grad + begin), V4, U4, groups,
                                [&](const float (&g)[4], const float (&v)[4], float (&u)[4], uint32_t o, auto&& next) {
      float a[4];
      accum4<kMom, kNest>(g, v, u, rule, a);
      next();
      stream_store<kNt>(V4 + o, vf4{a[0], a[1], a[2], a[3]});
      if constexpr (kMom) stream_store<kNt>(U4 + o, vf4{u[0], u[1], u[2], u[3]});
      f(a, 4u, begin + 4u * o);
    });
    base = begin + groups * kGroupElems;
  }
  for (; base < end; base += kGroupElems) {
    const uint32_t idx0 = base + lane * 4u;
    float g[4] = {0.f, 0.f, 0.f, 0.f}, v[4] = {0.f, 0.f, 0.f, 0.f}, u[4] = {0.f, 0.f, 0.f, 0.f}, a[4];
    const uint32_t nvalid = idx0 < end ? ((end - idx0) < 4u ? (end - idx0) : 4u) : 0u;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (static_cast<uint32_t>(j) < nvalid) {
        g[j] = G[idx0 + j];
        v[j] = V[idx0 + j];
        if constexpr (kMom) u[j] = U[idx0 + j];
      }
    }
    accum4<kMom, kNest>(g, v, u, rule, a);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (static_cast<uint32_t>(j) < nvalid) {
        V[idx0 + j] = a[j];
        if constexpr (kMom) U[idx0 + j] = u[j];
      }
    }
    f(a, nvalid, idx0);
  }
}

__device__ __forceinline__ float wave_max(float x) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) x = fmaxf(x, __shfl_xor(x, off));
  return x;
}

// The workgroup's elements above the threshold, from its waves' counts (every thread of a wave has its wave's).
__device__ __forceinline__ void leave_wg_count(const ThresholdArgs& A, uint32_t wg, uint32_t count, uint32_t* wave_counts) {
  if (lane_id() == 0u) wave_counts[threadIdx.x >> 6] = count;
  __syncthreads();
  if (threadIdx.x == 0u) {
    uint32_t sum = 0u;
#pragma unroll
    for (uint32_t w = 0; w < kWavesPerBlock; ++w) sum += wave_counts[w];
    A.wg_counts[wg] = sum;
  }
}

}  // namespace

// ------------------------------------------------------------------ sample (a search follows)
// One workgroup per layer, one piece of 16 consecutive elements a thread, each from a stretch of the layer of its own, and the
// magnitude that (4k of the layer's elements, and a margin for small samples) of them exceed, rounded down to 12 bits.
// Speed only: a magnitude that turns out too high or too low costs further passes, not the result.  (Scattered cache lines
// are what one workgroup waits for: 4096 pieces of four elements took 23 us on the LSTM set, these 14.5 us; counting only the
// samples above a bound, a fraction of the LDS atomics, changed nothing.)
__global__ void __launch_bounds__(kSampleThreads) threshold_sample_kernel(ThresholdArgs A) {
  __shared__ uint32_t hist[kHistBins];
  __shared__ uint32_t scan[kSampleThreads / kWaveSize];
  __shared__ uint32_t found;
  const uint32_t l = blockIdx.x, t = threadIdx.x;
  const LayerDesc L = A.layers[l];
  const uint32_t groups = (L.n + kPieceElems - 1u) / kPieceElems;
  const uint32_t pieces = threshold_sample_pieces(L.n);
  const unsigned long long rank = threshold_sample_rank(L.n, L.k);
  const bool listable = threshold_listable(L.n, L.k);
  for (uint32_t b = t; b < static_cast<uint32_t>(kHistBins); b += kSampleThreads) hist[b] = 0u;
  if (t == 0u) found = 0xFFFFFFFFu;
  __syncthreads();
  if (listable && t < pieces) {
    AccumRule rule;
    rule.m = A.m;
    rule.scale = A.grad_scale ? *as_global(A.grad_scale) : 1.0f;
    constexpr uint32_t kEach = kPieceElems / 4u;
    const uint32_t lo = static_cast<uint32_t>(static_cast<unsigned long long>(t) * groups / pieces);
    const uint32_t hi = static_cast<uint32_t>(static_cast<unsigned long long>(t + 1u) * groups / pieces);
    uint32_t h = (t + 1u) * 2654435761u;                     // (some place inside the stretch: rows of a matrix are not to line up)
    h ^= h >> 15; h *= 2246822519u; h ^= h >> 13;
    const uint32_t first = kPieceElems * (lo + static_cast<uint32_t>((static_cast<unsigned long long>(h) * (hi - lo)) >> 32));
    const uint32_t have = L.n - first < kPieceElems ? L.n - first : kPieceElems;
    float g[kEach][4], v[kEach][4], u[kEach][4];
#pragma unroll
    for (uint32_t q = 0; q < kEach; ++q) {
      const uint32_t e = first + 4u * q;
#pragma unroll
      for (int j = 0; j < 4; ++j) g[q][j] = v[q][j] = u[q][j] = 0.0f;
      if (4u * q + 4u <= have) {
        const vf4 gq = *as_vec(L.grad + e), vq = *as_vec(static_cast<const float*>(L.resid) + e);
        g[q][0] = gq.x; g[q][1] = gq.y; g[q][2] = gq.z; g[q][3] = gq.w;
        v[q][0] = vq.x; v[q][1] = vq.y; v[q][2] = vq.z; v[q][3] = vq.w;
        if (L.mom != nullptr) {
          const vf4 uq = *as_vec(static_cast<const float*>(L.mom) + e);
          u[q][0] = uq.x; u[q][1] = uq.y; u[q][2] = uq.z; u[q][3] = uq.w;
        }
      } else {
#pragma unroll
        for (uint32_t j = 0; j < 4u; ++j) {
          if (4u * q + j < have) {
            g[q][j] = as_global(L.grad)[e + j];
            v[q][j] = as_global(static_cast<const float*>(L.resid))[e + j];
            if (L.mom != nullptr) u[q][j] = as_global(static_cast<const float*>(L.mom))[e + j];
          }
        }
      }
    }
#pragma unroll
    for (uint32_t q = 0; q < kEach; ++q) {
      float a[4];
      if (L.mom == nullptr) accum4<false, false>(g[q], v[q], u[q], rule, a);
      else if (!A.nesterov) accum4<true, false>(g[q], v[q], u[q], rule, a);
      else accum4<true, true>(g[q], v[q], u[q], rule, a);
#pragma unroll
      for (uint32_t j = 0; j < 4u; ++j)
        if (4u * q + j < have && fabsf(a[j]) > 0.0f) atomicAdd(&hist[(fbits(a[j]) & kKeyMask) >> 19], 1u);
    }
  }
  __syncthreads();
  // four bins a thread, from the top
  uint32_t h[4], mine = 0u;
#pragma unroll
  for (uint32_t j = 0; j < 4u; ++j) { h[j] = hist[kHistBins - 1u - (4u * t + j)]; mine += h[j]; }
  uint32_t total;
  uint32_t cum = block_excl_scan<kSampleThreads / kWaveSize>(mine, scan, total);
  if (listable && cum < rank && rank <= cum + mine) {
#pragma unroll
    for (uint32_t j = 0; j < 4u; ++j) {
      if (cum < rank && rank <= cum + h[j]) found = kHistBins - 1u - (4u * t + j);
      cum += h[j];
    }
  }
  __syncthreads();
  if (t == 0u) {
    // (fewer non-zero samples than that: a sparse layer, every non-zero element is listed if they fit)
    const uint32_t bits = found != 0xFFFFFFFFu ? found << 19 : 0u;
    A.moments[l].listed_above = listable ? __uint_as_float(bits) : __uint_as_float(0x7F800000u);
  }
}

// ------------------------------------------------------------------ accumulate (+ moments, lists)
// Leaves in the wave-chunk's list the elements above a magnitude (as many as the list holds) and per wave-chunk their number;
// the magnitude is the threshold where it is given, and the sample's where it is searched (kSearch), in which case the pass
// also leaves per workgroup its part of the exactly rounded sum of |a| (rgc_exact.h) and the maximum of |a|.
template <bool kNt, bool kSearch, bool kReverse>
__global__ void __launch_bounds__(kBlockThreads) threshold_accumulate_kernel(ThresholdArgs A) {
  __shared__ ExactShared sh;
  __shared__ float wave_mx[kWavesPerBlock];
  __shared__ uint32_t wave_counts[kWavesPerBlock];
  if constexpr (kSearch) {
    exact_shared_init(sh);
    __syncthreads();
  }
  const uint32_t wg = (kReverse != (A.reverse != 0u)) ? gridDim.x - 1u - blockIdx.x : blockIdx.x;
  const uint32_t l = A.wg2layer[wg];
  const LayerDesc L = A.layers[l];
  const Place p = place_of(A, L, l, wg);
  ExactAcc acc{0.0, 0.0, 0u};
  float mx = 0.0f;
  uint32_t cnt = 0u;                        // elements above the magnitude so far, the same in every lane
  if (p.begin != p.end) {
    const float thr = !kSearch ? *as_global(A.thresholds + l) : A.sampled ? A.moments[l].listed_above : __uint_as_float(0x7F800000u);
    const gptr<vu2> slot = as_global(reinterpret_cast<vu2*>(A.slots + static_cast<size_t>(p.wc) * A.cap));
    auto take = [&](const float (&a)[4], uint32_t nvalid, uint32_t idx0) {
      if constexpr (kSearch) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          if (static_cast<uint32_t>(j) < nvalid) {
            const float mag = fabsf(a[j]);
            exact_add_f32(acc, mag, sh.digits);
            mx = fmaxf(mx, mag);
          }
        }
      }
      // the elements above the magnitude go to the wave-chunk's list in index order (ballot ranks);
      // a list that is full only counts on, and the later passes read that wave-chunk (or layer) from V instead
      bool f[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) f[j] = static_cast<uint32_t>(j) < nvalid && fabsf(a[j]) > thr;
      const unsigned long long m0 = __ballot(f[0]), m1 = __ballot(f[1]), m2 = __ballot(f[2]), m3 = __ballot(f[3]);
      if ((m0 | m1 | m2 | m3) == 0ull) return;
      uint32_t pos = cnt + rank_below(m0) + rank_below(m1) + rank_below(m2) + rank_below(m3);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (f[j]) {
          if (pos < A.cap) slot[pos] = vu2{fbits(a[j]), idx0 + static_cast<uint32_t>(j)};
          ++pos;
        }
      }
      cnt += popc64(m0) + popc64(m1) + popc64(m2) + popc64(m3);
    };
    AccumRule rule;
    rule.m = A.m;
    rule.scale = A.grad_scale ? *as_global(A.grad_scale) : 1.0f;
    if (L.mom == nullptr) accumulate_groups<kNt, false, false>(L, p.begin, p.end, rule, take);
    else if (!A.nesterov) accumulate_groups<kNt, true, false>(L, p.begin, p.end, rule, take);
    else accumulate_groups<kNt, true, true>(L, p.begin, p.end, rule, take);
    if (lane_id() == 0u) {
      A.counts[p.wc] = cnt;
      A.listed[p.wc] = cnt;
    }
  }
  if constexpr (kSearch) {
    const float m = wave_max(mx);
    if (lane_id() == 0u) wave_mx[threadIdx.x >> 6] = m;
    const ExactAcc total = exact_block_total(acc, sh);      // its barriers also order wave_mx
    if (threadIdx.x == 0u) {
      exact_store_part(A.sum_parts, wg, total, sh);
      float bm = wave_mx[0];
#pragma unroll
      for (int w = 1; w < kWavesPerBlock; ++w) bm = fmaxf(bm, wave_mx[w]);
      A.part_max[wg] = bm;
    }
  } else {
    leave_wg_count(A, wg, cnt, wave_counts);
  }
}

// ------------------------------------------------------------------ moments of a layer
// One workgroup per layer adds the parts of the layer's workgroups up, rounds the sum once, takes the
// maximum, stores mean, max and max - mean, and clears the layer's histogram for the pass that follows.
__global__ void __launch_bounds__(kBlockThreads) threshold_moments_kernel(ThresholdArgs A) {
  __shared__ ExactShared sh;
  __shared__ float wave_mx[kWavesPerBlock];
  __shared__ uint32_t scan[kWavesPerBlock];
  exact_shared_init(sh);
  __syncthreads();
  const uint32_t l = blockIdx.x;
  const LayerDesc L = A.layers[l];
  ExactPair acc;
  float mx = 0.0f;
  exact_take_parts(acc, A.sum_parts, L.wg_first, L.wg_count, sh);
  constexpr uint32_t kItems = 8;          // independent loads in flight per thread
  for (uint32_t base = threadIdx.x; base < L.wg_count; base += kItems * kBlockThreads) {
    float v[kItems];
#pragma unroll
    for (uint32_t j = 0; j < kItems; ++j) v[j] = base + j * kBlockThreads < L.wg_count ? A.part_max[L.wg_first + base + j * kBlockThreads] : 0.0f;
#pragma unroll
    for (uint32_t j = 0; j < kItems; ++j) mx = fmaxf(mx, v[j]);
  }
  // what the lists hold: all of them complete, and 2k elements or more together
  uint32_t listed = 0u, bad = 0u;
  for (uint32_t base = threadIdx.x; base < L.wc_count; base += kItems * kBlockThreads) {
    uint32_t v[kItems];
#pragma unroll
    for (uint32_t j = 0; j < kItems; ++j) v[j] = base + j * kBlockThreads < L.wc_count ? A.listed[L.wc_first + base + j * kBlockThreads] : 0u;
#pragma unroll
    for (uint32_t j = 0; j < kItems; ++j) { bad |= v[j] > A.cap ? 1u : 0u; listed += v[j]; }
  }
  uint32_t listed_all;
  (void)block_excl_scan(listed, scan, listed_all);
  bad = __syncthreads_or(static_cast<int>(bad)) ? 1u : 0u;
  mx = wave_max(mx);
  if (lane_id() == 0u) wave_mx[threadIdx.x >> 6] = mx;
  const double sum = exact_finish(acc, sh);                 // holds barriers
  if (threadIdx.x == 0u) {
    ThresholdMoments M;
    M.mean = static_cast<float>(sum / static_cast<double>(L.n));
    M.max = wave_mx[0];
#pragma unroll
    for (int w = 1; w < kWavesPerBlock; ++w) M.max = fmaxf(M.max, wave_mx[w]);
    M.span = __fsub_rn(M.max, M.mean);
    M.counts_taken = 0u;
    M.listed_above = A.sampled ? A.moments[l].listed_above : __uint_as_float(0x7F800000u);
    M.lists = !bad && listed_all >= 2u * L.k ? 1u : 0u;     // (k <= 2^30)
    A.moments[l] = M;
  }
  uint32_t* hist = A.hist + static_cast<size_t>(l) * kHistBins;
  for (uint32_t b = threadIdx.x; b < kHistReps * kSteps; b += kBlockThreads) hist[b] = 0u;
}

// ------------------------------------------------------------------ the threshold search (Section 2.1, Algorithm 3)
// The layer's histogram is complete; the number of elements above T(j) is the number of elements in the bins j .. 1023.
struct SearchShared {
  uint32_t above[kSteps + 1];
  uint32_t scan[kWavesPerBlock];
  uint32_t last;
};
__device__ __forceinline__ void search_threshold(const ThresholdArgs& A, uint32_t l, const LayerDesc& L, SearchShared& S) {
  uint32_t* hist = A.hist + static_cast<size_t>(l) * kHistBins;
  // suffix sums: thread t owns the bins 1023 - 4t and the three below (and leaves them zero: the exact path, which
  // shares the array, expects it cleared)
  constexpr uint32_t kPer = kSteps / kBlockThreads;
  uint32_t v[kHistReps][kPer], h[kPer], mine = 0u;
#pragma unroll
  for (uint32_t r = 0; r < kHistReps; ++r)
#pragma unroll
    for (uint32_t i = 0; i < kPer; ++i) v[r][i] = ld_agent(&hist[r * kSteps + kSteps - 1u - (threadIdx.x * kPer + i)]);
#pragma unroll
  for (uint32_t i = 0; i < kPer; ++i) {
    h[i] = 0u;
#pragma unroll
    for (uint32_t r = 0; r < kHistReps; ++r) {
      h[i] += v[r][i];
      hist[r * kSteps + kSteps - 1u - (threadIdx.x * kPer + i)] = 0u;
    }
    mine += h[i];
  }
  uint32_t total;
  uint32_t run = block_excl_scan(mine, S.scan, total);
#pragma unroll
  for (uint32_t i = 0; i < kPer; ++i) { run += h[i]; S.above[kSteps - 1u - (threadIdx.x * kPer + i)] = run; }
  __syncthreads();
  if (threadIdx.x == 0u) {
    // The search interval of Algorithm 3 starts as [0, 1] and is halved until it is 2^-10 wide, so its ends and
    // midpoints are the multiples j / 1024 and the bisection can run on the integers j: [lo, hi] starts as
    // [0, 1024], every midpoint is exact, and at most ten thresholds T(j) are tried.  More than k but fewer than
    // 2k elements above T(j) end the search; k or fewer mean the threshold has to come down (hi = j), otherwise up.
    ThresholdMoments M = A.moments[l];
    const unsigned long long k = L.k;
    uint32_t lo = 0u, hi = kSteps, counts = 0u;
    float thr = 0.0f;
    while (hi - lo > 1u) {
      const uint32_t j = lo + (hi - lo) / 2u;
      thr = threshold_at(M.mean, M.span, j);
      const unsigned long long nnz = S.above[j];
      ++counts;
      if (nnz > k && nnz < 2ull * k) break;
      if (nnz <= k) hi = j; else lo = j;
    }
    *as_global(A.thresholds + l) = thr;
    A.moments[l].counts_taken = counts;
    if (M.lists && thr < M.listed_above) A.moments[l].lists = 0u;   // (the lists know that 2k or more exceed it, not which)
  }
}

// ------------------------------------------------------------------ histogram over the candidate thresholds
// kHistReps copies of a layer's histogram: its workgroups mostly add to the same few bins, and atomics on one address take their
// turns (LSTM set, this launch 25.7 us with one copy, 20.6 with four, 28.3 with eight; VGG16 set, the call 671, 630, 637).
// The layer's last workgroup runs the search (as a launch
// of its own it took 5.4 us).
template <bool kReverse>
__global__ void __launch_bounds__(kBlockThreads) threshold_histogram_kernel(ThresholdArgs A) {
  __shared__ uint32_t lds_hist[kSteps];
  __shared__ SearchShared search;
  const uint32_t wg = (kReverse != (A.reverse != 0u)) ? gridDim.x - 1u - blockIdx.x : blockIdx.x;
  const uint32_t l = A.wg2layer[wg];
  const LayerDesc L = A.layers[l];
  const Place p = place_of(A, L, l, wg);
  for (uint32_t b = threadIdx.x; b < kSteps; b += kBlockThreads) lds_hist[b] = 0u;
  __syncthreads();
  const ThresholdMoments M = A.moments[l];
  const float inv = M.span > 0.0f ? static_cast<float>(kSteps) / M.span : 0.0f;
  uint32_t below = 0u;     // bin 0 is by far the fullest: counted in a register
  if (M.lists) for_listed(A, p, [&](const vu2& e, bool in) {
    const uint32_t b = in ? bin_of(fabsf(__uint_as_float(e.x)), M.mean, M.span, inv) : 0u;
    if (b != 0u) atomicAdd(&lds_hist[b], 1u);
    else below += in ? 1u : 0u;
  });
  else read_groups(L.resid, p.begin, p.end, [&](const float (&a)[4], uint32_t nvalid, uint32_t) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (static_cast<uint32_t>(j) < nvalid) {
        const uint32_t b = bin_of(fabsf(a[j]), M.mean, M.span, inv);
        if (b != 0u) atomicAdd(&lds_hist[b], 1u);
        else ++below;
      }
    }
  });
  if (below) atomicAdd(&lds_hist[0], below);
  __syncthreads();
  uint32_t* hist = A.hist + static_cast<size_t>(l) * kHistBins + (wg % kHistReps) * kSteps;
  for (uint32_t b = threadIdx.x; b < kSteps; b += kBlockThreads) {
    const uint32_t c = lds_hist[b];
    if (c) atomicAdd(&hist[b], c);
  }
  if (last_block_of_layer(&A.state[l].done, A.group_done + L.grp_first, wg - L.wg_first, L.wg_count, &search.last)) search_threshold(A, l, L, search);
}

// ------------------------------------------------------------------ count, offsets, emit
template <bool kReverse>
__global__ void __launch_bounds__(kBlockThreads) threshold_count_kernel(ThresholdArgs A) {
  const uint32_t wg = (kReverse != (A.reverse != 0u)) ? gridDim.x - 1u - blockIdx.x : blockIdx.x;
  const uint32_t l = A.wg2layer[wg];
  const LayerDesc L = A.layers[l];
  const Place p = place_of(A, L, l, wg);
  __shared__ uint32_t wave_counts[kWavesPerBlock];
  const float thr = *as_global(A.thresholds + l);
  uint32_t cnt = 0u;
  if (A.moments[l].lists) for_listed(A, p, [&](const vu2& e, bool in) { cnt += in && fabsf(__uint_as_float(e.x)) > thr ? 1u : 0u; });
  else read_groups(L.resid, p.begin, p.end, [&](const float (&a)[4], uint32_t nvalid, uint32_t) {
#pragma unroll
    for (int j = 0; j < 4; ++j) cnt += (static_cast<uint32_t>(j) < nvalid && fabsf(a[j]) > thr) ? 1u : 0u;
  });
  const uint32_t total = wave_total(wave_incl_scan(cnt));
  if (p.begin != p.end && lane_id() == 0u) A.counts[p.wc] = total;
  leave_wg_count(A, wg, total, wave_counts);
}

// Calls with a layer of more than kOffsetsWgs workgroups, one workgroup per layer: the wave-chunk counts become the wave-chunks' first
// output positions.  (By the last workgroup of the layer in the launch before: LSTM set 17.2 us instead of 4.6 + 4.6.)
__global__ void __launch_bounds__(kBlockThreads) threshold_offsets_kernel(ThresholdArgs A) {
  __shared__ uint32_t lds_scan[kWavesPerBlock];
  const uint32_t l = blockIdx.x;
  const LayerDesc L = A.layers[l];
  uint32_t* c = A.counts + L.wc_first;
  constexpr uint32_t kItems = 8;          // independent loads in flight per thread: this is a serial step
  uint32_t carry = 0u;
  for (uint32_t base = 0; base < L.wc_count; base += kBlockThreads * kItems) {
    const uint32_t i0 = base + threadIdx.x * kItems;
    uint32_t v[kItems], sum = 0u;
#pragma unroll
    for (uint32_t j = 0; j < kItems; ++j) {
      v[j] = (i0 + j < L.wc_count) ? c[i0 + j] : 0u;
      sum += v[j];
    }
    uint32_t total;
    uint32_t ex = carry + block_excl_scan(sum, lds_scan, total);
#pragma unroll
    for (uint32_t j = 0; j < kItems; ++j) {
      if (i0 + j < L.wc_count) c[i0 + j] = ex;
      ex += v[j];
    }
    carry += total;
  }
  if (threadIdx.x == 0u) {
    const uint32_t cap = 2u * L.k;
    *as_global(L.out_count) = static_cast<int32_t>(carry < cap ? carry : cap);
    if (A.nnz) *as_global(A.nnz + l) = static_cast<int32_t>(carry);
  }
}

// The accumulate pass of this call left the elements above the threshold (kSearch: those and others) in the wave-chunk
// lists; a wave-chunk whose list holds them all is written from it, without another look at V.
template <bool kReverse, bool kSearch>
__global__ void __launch_bounds__(kBlockThreads) threshold_emit_kernel(ThresholdArgs A) {
  const uint32_t wg = (kReverse != (A.reverse != 0u)) ? gridDim.x - 1u - blockIdx.x : blockIdx.x;
  const uint32_t l = A.wg2layer[wg];
  const LayerDesc L = A.layers[l];
  const Place p = place_of(A, L, l, wg);
  const uint32_t cap = 2u * L.k;
  uint32_t out_pos = p.begin != p.end ? A.counts[p.wc] : 0u;
  if (A.scanned == 0u) {
    // Where this wave's part of the message begins: every workgroup adds the counts of those before it up by itself, sixteen words of a
    // thread in flight.  (With one workgroup a layer and a launch for that instead, us per call, thresholds reused and searched: 66 M elements in
    // one tensor 165.9 / 157.5, 206.2 / 198.3, 134 M 315 / 294, 373 / 359, 400 M in four 915 / 879, 1044 / 1015.)
    __shared__ uint32_t sums[kWavesPerBlock], counts[kWavesPerBlock];
    const uint32_t wave = threadIdx.x >> 6, before = wg - L.wg_first;
    const gptr<const uint32_t> c = as_global(static_cast<const uint32_t*>(A.wg_counts)) + L.wg_first;
    constexpr uint32_t kItems = 16;
    uint32_t sum = 0u;
    for (uint32_t base = threadIdx.x; base < before; base += kItems * kBlockThreads) {
      uint32_t v[kItems];
#pragma unroll
      for (uint32_t j = 0; j < kItems; ++j) v[j] = base + j * kBlockThreads < before ? c[base + j * kBlockThreads] : 0u;
#pragma unroll
      for (uint32_t j = 0; j < kItems; ++j) sum += v[j];
    }
    sum = wave_total(wave_incl_scan(sum));
    if (lane_id() == 0u) { sums[wave] = sum; counts[wave] = out_pos; }
    __syncthreads();
    uint32_t first = 0u, all = 0u;
#pragma unroll
    for (uint32_t w = 0; w < kWavesPerBlock; ++w) {
      first += sums[w] + (w < wave ? counts[w] : 0u);
      all += sums[w] + counts[w];
    }
    out_pos = first;
    if (before + 1u == L.wg_count && threadIdx.x == 0u) {
      *as_global(L.out_count) = static_cast<int32_t>(all < cap ? all : cap);
      if (A.nnz) *as_global(A.nnz + l) = static_cast<int32_t>(all);
    }
  }
  if (p.begin == p.end) return;
  if (out_pos >= cap) return;                      // the buffer is full: the rest stays in the residual
  const bool clear_mom = (L.mom != nullptr) && A.mask_momentum;
  const gptr<int32_t> out_idx = as_global(L.out_idx);
  const gptr<float> out_val = as_global(L.out_val);
  const gptr<float> resid = as_global(L.resid);
  const gptr<float> mom = as_global(L.mom);
  if (kSearch ? A.moments[l].lists != 0u : A.listed[p.wc] <= A.cap) {
    const float above = *as_global(A.thresholds + l);
    for_listed(A, p, [&](const vu2& e, bool in) {
      const bool sel = in && fabsf(__uint_as_float(e.x)) > above;
      const unsigned long long m = __ballot(sel);
      const uint32_t pos = out_pos + rank_below(m);
      if (sel && pos < cap) {
        out_idx[pos] = static_cast<int32_t>(e.y);
        out_val[pos] = __uint_as_float(e.x);
        mask_store(resid + e.y);
        if (clear_mom) mask_store(mom + e.y);
      }
      out_pos += popc64(m);
    });
    return;
  }
  const float thr = *as_global(A.thresholds + l);
  read_groups(L.resid, p.begin, p.end, [&](const float (&a)[4], uint32_t nvalid, uint32_t idx0) {
    bool sel[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) sel[j] = static_cast<uint32_t>(j) < nvalid && fabsf(a[j]) > thr;
    const unsigned long long s0 = __ballot(sel[0]), s1 = __ballot(sel[1]), s2 = __ballot(sel[2]), s3 = __ballot(sel[3]);
    if ((s0 | s1 | s2 | s3) == 0ull) return;
    uint32_t pos = out_pos + rank_below(s0) + rank_below(s1) + rank_below(s2) + rank_below(s3);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (sel[j]) {
        if (pos < cap) {
          out_idx[pos] = static_cast<int32_t>(idx0 + j);
          out_val[pos] = a[j];
          mask_store(resid + idx0 + j);
          if (clear_mom) mask_store(mom + idx0 + j);
        }
        ++pos;
      }
    }
    out_pos += popc64(s0) + popc64(s1) + popc64(s2) + popc64(s3);
  });
}

hipError_t launch_threshold_compress(const ThresholdArgs& a, uint32_t num_wgs, uint32_t num_layers, hipStream_t s) {
  const dim3 block(kBlockThreads);
#define RGC_LAUNCHED() do { hipError_t e_ = hipGetLastError(); if (e_ != hipSuccess) return e_; } while (0)
  // Each pass over the tensors runs against the direction of the one before it: what that one touched last
  // (still in the memory-side cache) is read first.  a.reverse turns the whole sequence round.
  if (a.search) {
    if (a.sampled) {
      hipLaunchKernelGGL(threshold_sample_kernel, dim3(num_layers), dim3(kSampleThreads), 0, s, a);
      RGC_LAUNCHED();
    }
    if (a.past_cache) hipLaunchKernelGGL((threshold_accumulate_kernel<true, true, false>), dim3(num_wgs), block, 0, s, a);
    else hipLaunchKernelGGL((threshold_accumulate_kernel<false, true, false>), dim3(num_wgs), block, 0, s, a);
    RGC_LAUNCHED();
    hipLaunchKernelGGL(threshold_moments_kernel, dim3(num_layers), block, 0, s, a);
    RGC_LAUNCHED();
    hipLaunchKernelGGL(threshold_histogram_kernel<true>, dim3(num_wgs), block, 0, s, a);
    RGC_LAUNCHED();
    hipLaunchKernelGGL(threshold_count_kernel<false>, dim3(num_wgs), block, 0, s, a);
    RGC_LAUNCHED();
    if (a.scanned) hipLaunchKernelGGL(threshold_offsets_kernel, dim3(num_layers), block, 0, s, a);
    RGC_LAUNCHED();
    hipLaunchKernelGGL((threshold_emit_kernel<true, true>), dim3(num_wgs), block, 0, s, a);
  } else {
    if (a.past_cache) hipLaunchKernelGGL((threshold_accumulate_kernel<true, false, false>), dim3(num_wgs), block, 0, s, a);
    else hipLaunchKernelGGL((threshold_accumulate_kernel<false, false, false>), dim3(num_wgs), block, 0, s, a);
    RGC_LAUNCHED();
    if (a.scanned) hipLaunchKernelGGL(threshold_offsets_kernel, dim3(num_layers), block, 0, s, a);
    RGC_LAUNCHED();
    hipLaunchKernelGGL((threshold_emit_kernel<true, false>), dim3(num_wgs), block, 0, s, a);
  }
#undef RGC_LAUNCHED
  return hipGetLastError();
}

}  // namespace rgc
