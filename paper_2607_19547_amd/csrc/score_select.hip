// Per-token key deviation (Eq. 5) and deterministic top-k selection.
//
// delta_t = || k_fresh[:, t - s1, :] - k[score_layer][:, t, :] ||_2 over all
// KV heads x head_dim, accumulated in float64 (bf16 differences and their
// squares are exact in float64) and rounded once to float32.
//
// Selection ranks the float32 scores.  Scores are >= 0, so their IEEE bit
// patterns order like integers.  Up to 512 candidates each score is ranked
// against every other; beyond that a radix select (11 + 11 + 9 bits) finds the
// k-th largest pattern.  Either way the taken scores (every one above the
// threshold and the lowest-index ties at it) are compacted in index order, so
// the output is ascending and exactly k long.  All counts are order
// independent, so the result is deterministic.
#include <type_traits>

#include "cs_common.h"

namespace cs {

template <typename E>
__device__ __forceinline__ double ldd(const E* p);
template <>
__device__ __forceinline__ double ldd<float>(const float* p) { return (double)*p; }
template <>
__device__ __forceinline__ double ldd<uint16_t>(const uint16_t* p) { return (double)bf16_to_f32(*p); }

// One wavefront per candidate token.  Rows of the score layer are reached
// through the cache's row map (plane = score_layer * H_kv + head).
template <typename E, typename Rows>
__global__ __launch_bounds__(256) void deviation_score(const Rows rows, const E* __restrict__ kf,
                                                       float* __restrict__ scores, int score_layer,
                                                       int64_t n, int64_t cs1, int Hkv, int D) {
  const int64_t tok = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (tok >= n) return;  // whole wavefront
  const int lane = threadIdx.x & 63;
  double acc = 0.0;
  for (int h = 0; h < Hkv; ++h) {
    const E* a = (const E*)rows.row(false, (int64_t)score_layer * Hkv + h, cs1 + tok, D * (int)sizeof(E));
    const E* b = kf + ((int64_t)h * n + tok) * D;
    for (int d = lane; d < D; d += 64) {
      const double x = ldd(b + d) - ldd(a + d);
      acc = fma(x, x, acc);
    }
  }
#pragma unroll
  for (int o = 32; o; o >>= 1) acc += __shfl_xor(acc, o);
  if (lane == 0) scores[tok] = (float)sqrt(acc);
}

// bf16, D = 128: 16 lanes per token, 8 elements per lane per head.
template <typename Rows>
__global__ __launch_bounds__(256) void deviation_score_bf16_d128(const Rows rows, const uint16_t* __restrict__ kf,
                                                                 float* __restrict__ scores, int score_layer,
                                                                 int64_t n, int64_t cs1, int Hkv) {
  const int64_t tok = (int64_t)blockIdx.x * 16 + (threadIdx.x >> 4);
  const int j = threadIdx.x & 15;
  double acc = 0.0;
  if (tok < n) {
    for (int h = 0; h < Hkv; ++h) {
      const u32x4 a = *(const u32x4*)((const uint16_t*)rows.row(false, (int64_t)score_layer * Hkv + h, cs1 + tok, 256) + 8 * j);
      const u32x4 b = *(const u32x4*)(kf + ((int64_t)h * n + tok) * 128 + 8 * j);
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const double x0 = (double)bf16_lo(b[w]) - (double)bf16_lo(a[w]);
        const double x1 = (double)bf16_hi(b[w]) - (double)bf16_hi(a[w]);
        acc = fma(x0, x0, acc);
        acc = fma(x1, x1, acc);
      }
    }
  }
#pragma unroll
  for (int o = 8; o; o >>= 1) acc += __shfl_xor(acc, o, 16);
  if (tok < n && j == 0) scores[tok] = (float)sqrt(acc);
}

// ------------------------------------------------------------------ selection
constexpr int kSelThreads = 1024;
constexpr int kSelWaves = kSelThreads / 64;
constexpr int kSelGroup = 256;     // scores a wavefront takes at a time, four consecutive ones per lane
constexpr int kSelBatch = 8;       // groups in flight per wavefront
constexpr int kSelParts = 8;       // workgroups that share the compaction, at most
constexpr int kSelBins = 8192;     // first digit: exponent and five mantissa bits
constexpr int kSelShift = 18;      // bits below it
constexpr int kSelCopies = 2;      // copies of its histogram, by lane
constexpr int kSelSample = 8192;   // scores sampled, at most
constexpr int kSelList = 20480;    // scores of the band kept in LDS, at most
constexpr int kSegBits = 7;        // a list entry is (score - band start) << kSegBits | segment
static_assert(kSelWaves * kSelParts == 1 << kSegBits, "segment numbers fit their field");
constexpr int kRankMax = 512;      // candidates up to which every score is ranked against every other

// Few candidates (n <= kRankMax, one thread each): a score's rank is the
// number of scores above it plus the equal ones before it; ranks below k are
// taken.  One pass and three barriers, where the radix select below would
// spend its time on clearing and scanning bins (32 candidates: 2.4 against
// 27 us for the four-pass form it replaced).
__global__ __launch_bounds__(kRankMax) void rank_select_topk(const float* __restrict__ scores, int n, int k, int cs1,
                                                             int32_t* __restrict__ sel) {
  __shared__ __attribute__((aligned(16))) int val[kRankMax];
  __shared__ int taken[kRankMax / 64];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  // scores are >= 0: their patterns order like the signed integers they are;
  // threads past n hold -1, below every score
  // (the sign of a NaN is dropped: every score counts)
  const int u = tid < n ? ((const int*)scores)[tid] & 0x7fffffff : -1;
  val[tid] = u;
  __syncthreads();
  int rank = 0;
  const int n4 = (n + 3) >> 2, lo4 = 16 * wave, hi4 = min(n4, lo4 + 16);
  const int4* v4 = (const int4*)val;
#pragma unroll 4
  for (int j = 0; j < lo4; ++j) {  // every index here is below this wavefront's
    const int4 x = v4[j];
    rank += (x.x >= u) + (x.y >= u) + (x.z >= u) + (x.w >= u);
  }
  for (int j = lo4; j < hi4; ++j) {
    const int4 x = v4[j];
    rank += (x.x > u || (x.x == u && 4 * j < tid)) + (x.y > u || (x.y == u && 4 * j + 1 < tid)) +
            (x.z > u || (x.z == u && 4 * j + 2 < tid)) + (x.w > u || (x.w == u && 4 * j + 3 < tid));
  }
#pragma unroll 4
  for (int j = hi4; j < n4; ++j) {
    const int4 x = v4[j];
    rank += (x.x > u) + (x.y > u) + (x.z > u) + (x.w > u);
  }
  const bool take = tid < n && rank < k;
  const unsigned long long m = __ballot(take);
  if (lane == 0) taken[wave] = __popcll(m);
  __syncthreads();
  int pos = __popcll(m & ((1ull << lane) - 1ull));
  for (int w = 0; w < wave; ++w) pos += taken[w];
  if (take && pos < k) sel[pos] = cs1 + tid;
}

// A histogram of kBins bins in kCopies copies: bin d's copies start at word
// hist_at(d).  Thread t of a scan reads `per` bins side by side; two words of
// padding after every eight spread those reads over the banks.
template <int kBins, int kCopies>
__device__ __forceinline__ constexpr unsigned hist_at(unsigned d) {
  return kBins > kSelThreads * 2 ? d * kCopies + 2 * (d >> 3) : d * kCopies;
}

// The digits of the kk[i]-th largest scores (kRanks of them, in LDS order): the
// highest bin at which the count of scores in it and above reaches kk.  res[i]
// = {digit, kk less the scores above it, scores in it}.  Thread t takes `per`
// bins in descending order.
struct Digit {
  unsigned digit, left, in;
};
template <int kBins, int kCopies, int kRanks>
__device__ __forceinline__ void find_digits(const unsigned* hist, const unsigned (&kk)[kRanks], unsigned* tot,
                                            Digit* res) {
  constexpr int per = kBins > kSelThreads ? kBins / kSelThreads : 1;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  unsigned c[per], x = 0;
#pragma unroll
  for (int i = 0; i < per; ++i) {
    const int d = kBins - 1 - per * tid - i;
    c[i] = 0;
    if (d >= 0) {
#pragma unroll
      for (int y = 0; y < kCopies; ++y) c[i] += hist[hist_at<kBins, kCopies>((unsigned)d) + y];
    }
    x += c[i];
  }
  unsigned p = wave_scan(x);
  if (lane == 63) tot[wave] = p;
  __syncthreads();
  const unsigned t = lane < wave ? tot[lane & (kSelWaves - 1)] : 0u;  // (wave < 16)
  p += (unsigned)__builtin_amdgcn_readlane((int)wave_scan(t), 63);
#pragma unroll
  for (int r = 0; r < kRanks; ++r) {
    unsigned above = p - x;
    if (above < kk[r] && kk[r] <= p) {
      int i = 0;
#pragma unroll
      for (int j = 0; j < per - 1; ++j)
        if (i == j && above + c[j] < kk[r]) {
          above += c[j];
          ++i;
        }
      unsigned cnt = c[0];
#pragma unroll
      for (int j = 1; j < per; ++j)
        if (i == j) cnt = c[j];
      res[r] = {(unsigned)(kBins - 1 - per * tid - i), kk[r] - above, cnt};
    }
  }
  __syncthreads();
}
template <int kBins, int kCopies>
__device__ __forceinline__ void find_digit(const unsigned* hist, unsigned kk, unsigned* tot, Digit* res) {
  const unsigned one[1] = {kk};
  find_digits<kBins, kCopies, 1>(hist, one, tot, res);
}

// Selection of the k largest of n scores, in index order.  Every workgroup of
// the launch finds the same threshold; each then writes its share of the
// output (gridDim.x of them, at most kSelParts), so nothing passes between
// workgroups and no scratch memory is needed.
//
// A wavefront owns `ng` consecutive groups of 256 scores, split into gridDim.x
// equal segments; workgroup b compacts segment b of every wavefront.
//  1. A histogram of a sample (one score from every `stride` consecutive ones,
//     at a scattered place) brackets the k-th largest score: the band runs
//     from the sample's rank k S / n + delta to the rank k S / n - delta, with
//     delta four standard deviations.  Up to 8,192 scores the sample is all
//     of them and the band is one bin.
//  2. One pass over the scores counts those above the band, per segment, and
//     gathers the band (a few per cent) into LDS.
//  3. A radix select over the list finds the threshold.
//  4. Each workgroup writes its segments in one more partial pass.
// If the band misses the k-th score or overflows the list, a histogram of all
// scores and passes over memory for the lower digits take the place of 1 to 3.
//
// Bound: one CU's vector instructions, about ten per score in pass 2 (29 us of
// the 46-50 us that 260,096 scores take; 8 of 16 us for 63,488).  A histogram of
// every score instead (an LDS add of 64 scores takes more than ten
// instructions) and passes over memory for the lower digits take 102 us for
// 260,096; the four-digit form with a histogram per wavefront and one load in
// flight, which this replaced, took 335 us (48 us for 63,488, held in
// registers).  A band that holds more than the list (scores of which many
// per cent lie within a few per cent of the k-th) is found out by pass 2, and
// the histogram comes on top; from about 340,000 candidates at k = n / 2 (490,000
// at n / 10) on the list is too short for the sample's band, and the histogram
// comes at once.  Score and selection together, one head of D = 2, 260,096
// candidates, k = n / 10: 100 us for log-normal scores, 209 for norms of 256
// normal draws, 230 for equal scores; 500,000 candidates 299, 336, 580 (the form
// replaced: 386, 313, 334; 735, 598, 641).
__global__ __launch_bounds__(kSelThreads) void radix_select_topk(const float* __restrict__ scores, int n, int k,
                                                                 int cs1, int ng, int32_t* __restrict__ sel) {
  constexpr int kHist = kSelBins * kSelCopies + kSelBins / 4;  // words of the first digit's histogram, padding included
  __shared__ __attribute__((aligned(16))) unsigned hist[kHist];
  __shared__ unsigned list[kSelList + 64];  // (the last 64 take the writes of lanes with nothing to list)
  __shared__ unsigned seg[kSelWaves * kSelParts];  // taken scores per segment
  __shared__ unsigned tot[kSelWaves], eqs[kSelWaves];
  __shared__ Digit res[2];
  __shared__ unsigned s_list, s_above;
  __shared__ int s_cut;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int parts = gridDim.x, part = blockIdx.x;
  const int gp = ng / parts;  // groups per segment
  const unsigned* bits = (const unsigned*)scores;

  // f(four scores, index of the first) over groups [g0, g1) of this
  // wavefront, kSelBatch groups of loads in flight, b(...) after each batch;
  // scores past n are 0xffffffff, the others have the sign bit clear (also a
  // NaN: every score counts, so a digit is always found)
  auto load = [&](u32x4* u, int g, int g1) {
    // (uniform branches only, so that every load is issued before the first wait)
    const unsigned first = (unsigned)(wave * ng + g) * kSelGroup, last = (unsigned)n;
#pragma unroll
    for (int j = 0; j < kSelBatch; ++j) {
      const unsigned i0 = first + j * kSelGroup, i = i0 + 4 * lane;
      u[j] = u32x4{0xffffffffu, 0xffffffffu, 0xffffffffu, 0xffffffffu};
      if (g + j < g1) {
        if (i0 + kSelGroup <= last) {
          u[j] = *(const u32x4*)(bits + i);
        } else if (i0 < last) {
#pragma unroll
          for (int e = 0; e < 4; ++e) u[j][e] = bits[min(i + e, last - 1u)];
        }
      }
    }
#pragma unroll
    for (int j = 0; j < kSelBatch; ++j) {
      const unsigned i0 = first + j * kSelGroup, i = i0 + 4 * lane;
      if (g + j < g1 && i0 < last) {
#pragma unroll
        for (int e = 0; e < 4; ++e) u[j][e] &= 0x7fffffffu;
        if (i0 + kSelGroup > last) {
#pragma unroll
          for (int e = 0; e < 4; ++e) u[j][e] = i + e < last ? u[j][e] : 0xffffffffu;
        }
      }
    }
  };
  auto visit = [&](int g0, int g1, auto f) {
    for (int g = g0; g < g1; g += kSelBatch) {
      u32x4 u[kSelBatch];
      const unsigned first = (unsigned)(wave * ng + g) * kSelGroup;
      if (first >= (unsigned)n) break;  // (uniform)
      load(u, g, g1);
#pragma unroll
      for (int j = 0; j < kSelBatch; ++j)
        if (g + j < g1 && first + j * kSelGroup < (unsigned)n)  // (uniform)
          f(u[j], (int)(first + j * kSelGroup + 4 * lane), g + j);
    }
  };
  auto clear = [&](int words) {
    for (int b = tid; b < words / 4; b += kSelThreads) ((u32x4*)hist)[b] = u32x4{0u, 0u, 0u, 0u};
  };
  const int copy = lane & (kSelCopies - 1);
  // Whether a group's scores are all alike from bit `shift` up (*d0), so that one
  // add counts them: adds to one bin go through one by one.  Asked only where
  // every score sampled has the same first digit (260,096 equal scores: 230 us
  // with it, 340 without).
  bool crowded = false;
  auto one_digit = [&](const u32x4& u, int shift, unsigned* d0) -> bool {
    *d0 = (unsigned)__builtin_amdgcn_readfirstlane((int)(u[0] >> shift));  // (lane 0 holds a score)
    bool same = true;
#pragma unroll
    for (int e = 0; e < 4; ++e) same &= u[e] >> shift == *d0;
    return __ballot(same) == ~0ull;
  };

  // 1. the sample and the band [lo, hi)
  const int stride = (n + kSelSample - 1) / kSelSample, ns = (n + stride - 1) / stride;
  const float p = (float)k / (float)n;
  const int delta = stride == 1 ? 0 : (int)(4.f * sqrtf((float)ns * p * (1.f - p))) + 4;
  bool listed = (float)n * (2.f * (float)delta / (float)ns + 0.015f) <= (float)kSelList || stride == 1;
  clear(kHist);
  if (tid < kSelWaves * kSelParts) seg[tid] = 0;
  if (tid == 0) {
    s_list = 0;
    s_above = 0;
    s_cut = 0x7fffffff;
  }
  __syncthreads();
  unsigned thr = 0;           // the k-th largest score,
  unsigned kk = 0, ties = 0;  // how many scores equal to it are taken, how many there are (in the list)
  unsigned lo = 0;
  if (listed) {
    unsigned v[kSelSample / kSelThreads];
#pragma unroll
    for (int j = 0; j < kSelSample / kSelThreads; ++j) {
      const unsigned t = tid + j * kSelThreads;
      const unsigned jit = (unsigned)(((unsigned long long)(t * 2654435761u) * (unsigned)stride) >> 32);
      v[j] = bits[min((unsigned long long)t * (unsigned)stride + jit, (unsigned long long)(n - 1))];
    }
#pragma unroll
    for (int j = 0; j < kSelSample / kSelThreads; ++j)
      if (tid + j * kSelThreads < ns)
        atomicAdd(&hist[hist_at<kSelBins, kSelCopies>((v[j] & 0x7fffffffu) >> kSelShift) + copy], 1u);
    __syncthreads();
    const int r = (int)((float)ns * p + 0.5f);
    const int r_hi = stride == 1 ? k : max(1, r - delta), r_lo = stride == 1 ? k : max(r_hi, min(ns - 1, r + delta));
    const unsigned ranks[2] = {(unsigned)r_hi, (unsigned)r_lo};
    find_digits<kSelBins, kSelCopies, 2>(hist, ranks, tot, res);
    crowded = res[0].in == (unsigned)ns;
    unsigned hi = (res[0].digit + 1u) << kSelShift;
    lo = res[1].digit << kSelShift;
    // the band's width fits a list entry, and it reaches past the sample's
    // ends where the rank does
    const unsigned most = 1u << (32 - kSegBits);
    if (stride > 1 && r_hi == 1) hi = min(lo + most, 0x80000000u);
    if (stride > 1 && r_lo >= ns - 1) lo = hi > most ? hi - most : 0u;
    const unsigned span = min(hi - lo, most);
    hi = lo + span;
    // 2. scores above the band per segment, the band's scores into the list
    int s = wave * parts, rem = gp;  // segment of the next group, groups left in it
    unsigned above = 0, above_all = 0;
    for (int g = 0; g < ng; g += kSelBatch) {
      if ((unsigned)(wave * ng + g) * kSelGroup >= (unsigned)n) break;  // (uniform)
      u32x4 u[kSelBatch];
      load(u, g, ng);
      unsigned c = 0;
      int s1 = s, rem1 = rem;
#pragma unroll
      for (int j = 0; j < kSelBatch; ++j) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          above += __popcll(__ballot((int)u[j][e] > (int)(hi - 1u)));  // (0xffffffff is below)
          c += u[j][e] - lo < span;
        }
        if (--rem1 == 0) {  // (uniform)
          if (lane == 0 && s1 < (wave + 1) * parts) seg[s1] = above;
          above_all += above;
          above = 0;
          rem1 = gp;
          ++s1;
        }
      }
      const unsigned before = wave_scan(c), all = (unsigned)__builtin_amdgcn_readlane((int)before, 63);
      unsigned base = 0;
      if (lane == 0) base = atomicAdd(&s_list, all);
      base = (unsigned)__builtin_amdgcn_readfirstlane((int)base);
      unsigned at = base + before - c;
      const bool room = base + all <= kSelList;  // (uniform; past it the count alone matters)
#pragma unroll
      for (int j = 0; j < kSelBatch; ++j) {
        // (no branches: a band of a few per cent leaves few wavefronts without a write)
        if (room) {
          const unsigned off = (unsigned)s - (lo << kSegBits);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const bool in = u[j][e] - lo < span;
            list[in ? at : kSelList + lane] = (u[j][e] << kSegBits) + off;
            at += in;
          }
        }
        if (--rem == 0) {
          rem = gp;
          ++s;
        }
      }
    }
    if (lane == 0) {
      if (above) seg[s] = above;
      if (above + above_all) atomicAdd(&s_above, above + above_all);
    }
    clear(2048);
    __syncthreads();
    const unsigned m = s_list, over = s_above;
    listed = m <= kSelList && (unsigned)k > over && (unsigned)k - over <= m;  // the threshold is in the list
    if (listed) {
      // 3. radix select over the list, 11 bits at a time from the band's width
      kk = (unsigned)k - over;
      int shift = 32 - __builtin_clz(max(span - 1u, 1u));
      unsigned pre = 0;  // the threshold's bits at and above `shift`
      while (shift > 0) {
        const int w = min(shift, 11);
        const int up = shift;
        shift -= w;
        for (int j = tid; j < (int)m; j += kSelThreads) {
          const unsigned d = list[j] >> kSegBits;
          if (d >> up == pre) atomicAdd(&hist[(d >> shift) & ((1u << w) - 1u)], 1u);
        }
        __syncthreads();
        find_digit<2048, 1>(hist, kk, tot, res);
        pre = pre << w | res[0].digit;
        kk = res[0].left;
        ties = res[0].in;
        clear(2048);
        __syncthreads();
      }
      thr = lo + pre;
    }
  }
  if (!listed) {
    // every score: first digit, then the 18 bits below it as 11 and 7
    __syncthreads();
    clear(kHist);
    if (tid < kSelWaves * kSelParts) seg[tid] = 0;
    __syncthreads();
    // (two loops each: a test in the usual one costs it 5%)
    auto first_digits = [&](auto alike) {
      visit(0, ng, [&](const u32x4& u, int, int) {
        if constexpr (decltype(alike)::value) {
          unsigned d0;
          if (one_digit(u, kSelShift, &d0)) {
            if (lane == 0) atomicAdd(&hist[hist_at<kSelBins, kSelCopies>(d0)], (unsigned)kSelGroup);
            return;
          }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if ((int)u[e] >= 0) atomicAdd(&hist[hist_at<kSelBins, kSelCopies>(u[e] >> kSelShift) + copy], 1u);
      });
    };
    if (crowded) first_digits(std::true_type{});  // (uniform)
    else first_digits(std::false_type{});
    __syncthreads();
    find_digit<kSelBins, kSelCopies>(hist, (unsigned)k, tot, res);
    thr = res[0].digit;
    kk = res[0].left;
    int below = kSelShift;
    while (below > 0) {
      const int w = min(below, 11), up = below;
      below -= w;
      clear(2048 * 8);
      __syncthreads();
      auto lower_digits = [&](auto alike) {
        visit(0, ng, [&](const u32x4& u, int, int) {
          if constexpr (decltype(alike)::value) {
            unsigned d0;
            if (one_digit(u, below, &d0)) {
              if (lane == 0 && d0 >> w == thr) atomicAdd(&hist[(d0 & ((1u << w) - 1u)) * 8], (unsigned)kSelGroup);
              return;
            }
          }
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (u[e] >> up == thr) atomicAdd(&hist[((u[e] >> below) & ((1u << w) - 1u)) * 8 + (lane & 7)], 1u);
        });
      };
      if (crowded) lower_digits(std::true_type{});
      else lower_digits(std::false_type{});
      __syncthreads();
      find_digit<2048, 8>(hist, kk, tot, res);
      thr = thr << w | res[0].digit;
      kk = res[0].left;
      ties = res[0].in;
      __syncthreads();  // (res is written again)
    }
  }
  // the last tie that is taken, by index
  if (kk < ties) {  // (uniform)
    unsigned c = 0;
    visit(0, ng, [&](const u32x4& u, int, int) {
#pragma unroll
      for (int e = 0; e < 4; ++e) c += __popcll(__ballot(u[e] == thr));
    });
    if (lane == 0) eqs[wave] = c;
    __syncthreads();
    unsigned before = 0;
    for (int w = 0; w < wave; ++w) before += eqs[w];
    if (before < kk && kk <= before + c) {  // (uniform) the cut lies in this wavefront's range
      visit(0, ng, [&](const u32x4& u, int i, int) {
        unsigned rank = before;  // ties before this lane's first score
        unsigned all = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const unsigned long long m = __ballot(u[e] == thr);
          rank += __popcll(m & ((1ull << lane) - 1ull));
          all += __popcll(m);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (u[e] == thr && ++rank == kk) s_cut = i + e;
        before += all;
      });
    }
  }
  __syncthreads();
  const int cut = s_cut;
  auto taken = [&](unsigned u, int i) { return (int)u > (int)thr || (u == thr && i <= cut); };
  // taken scores per segment
  if (listed && kk == ties) {  // every tie: the list tells
    const unsigned d_thr = thr - lo;
    for (int j = tid; j < (int)s_list; j += kSelThreads)
      if (list[j] >> kSegBits >= d_thr) atomicAdd(&seg[list[j] & (kSelWaves * kSelParts - 1)], 1u);
  } else {
    if (tid < kSelWaves * kSelParts) seg[tid] = 0;
    __syncthreads();
    visit(0, ng, [&](const u32x4& u, int i, int g) {
      unsigned c = 0;
#pragma unroll
      for (int e = 0; e < 4; ++e) c += __popcll(__ballot(taken(u[e], i + e)));
      if (lane == 0) atomicAdd(&seg[wave * parts + g / gp], c);
    });
  }
  __syncthreads();
  // 4. this workgroup's segment of every wavefront, in index order
  const int mine = wave * parts + part;
  unsigned pos = 0;
#pragma unroll
  for (int s = 0; s < kSelWaves * kSelParts; s += 64)
    if (s + lane < mine) pos += seg[s + lane];
#pragma unroll
  for (int o = 32; o; o >>= 1) pos += __shfl_xor(pos, o);
  visit(part * gp, (part + 1) * gp, [&](const u32x4& u, int i, int) {
    unsigned at = pos, all = 0;
    bool t[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      t[e] = taken(u[e], i + e);
      const unsigned long long m = __ballot(t[e]);
      at += __popcll(m & ((1ull << lane) - 1ull));
      all += __popcll(m);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (t[e]) {
        if (at < (unsigned)k) sel[at] = cs1 + i + e;
        ++at;
      }
    pos += all;
  });
}

// Groups per wavefront and workgroups of the selection's launch: segments of
// at least two groups, at most kSelParts workgroups.
static void radix_shape(int64_t n, int* ng, int* parts) {
  const int64_t per = (n + kSelGroup * kSelWaves - 1) / (kSelGroup * kSelWaves);
  int p = 1;
  while (p < kSelParts && 4 * p <= per) p *= 2;
  *parts = p;
  *ng = (int)((per + p - 1) / p * p);
}

template <typename Rows>
static void launch_score(const Geo& g, const Rows& rows, int score_layer, const void* k_fresh, float* scores,
                         hipStream_t s) {
  static_assert(sizeof(Rows) + 64 <= 4096, "kernel arguments within 4 KB");
  TraceScope tr("deviation_score", s);
  if (g.dtype == CS_BF16 && g.D == 128) {
    const int64_t blocks = (g.n + 15) / 16;
    CS_LAUNCH(tr, deviation_score_bf16_d128<Rows>, dim3((unsigned)blocks), dim3(256), 0, s, rows,
                       (const uint16_t*)k_fresh, scores, score_layer, g.n, g.cs1, g.Hkv);
  } else {
    const int64_t blocks = (g.n + 3) / 4;
    if (g.dtype == CS_BF16)
      CS_LAUNCH(tr, (deviation_score<uint16_t, Rows>), dim3((unsigned)blocks), dim3(256), 0, s, rows,
                         (const uint16_t*)k_fresh, scores, score_layer, g.n, g.cs1, g.Hkv, g.D);
    else
      CS_LAUNCH(tr, (deviation_score<float, Rows>), dim3((unsigned)blocks), dim3(256), 0, s, rows,
                         (const float*)k_fresh, scores, score_layer, g.n, g.cs1, g.Hkv, g.D);
  }
}

cs_status launch_score_select(const Geo& g, const CacheView& cv, int score_layer, const void* k_fresh, float* scores,
                              int32_t* sel, int64_t k_sel, hipStream_t s, bool check_only) {
  const bool fast = g.dtype == CS_BF16 && g.D == 128;
  cs_status st0 = check_grid(fast ? (g.n + 15) / 16 : (g.n + 3) / 4, 1, 1, 256, "deviation score");
  if (st0 || check_only) return st0;
  if (cv.paged) launch_score(g, cv.pages<kMaxPages>(g), score_layer, k_fresh, scores, s);
  else launch_score(g, cv.flat(g), score_layer, k_fresh, scores, s);
  cs_status st = check_launch("deviation score launch");
  if (st || k_sel == 0) return st;
  {
    TraceScope tr(g.n <= kRankMax ? "rank_select_topk" : "radix_select_topk", s);
    if (g.n <= kRankMax) {
      CS_LAUNCH(tr, rank_select_topk, dim3(1), dim3((unsigned)((g.n + 63) / 64 * 64)), 0, s, scores, (int)g.n,
                (int)k_sel, (int)g.cs1, sel);
    } else {
      int ng, parts;
      radix_shape(g.n, &ng, &parts);
      CS_LAUNCH(tr, radix_select_topk, dim3(parts), dim3(kSelThreads), 0, s, scores, (int)g.n, (int)k_sel,
                (int)g.cs1, ng, sel);
    }
  }
  return check_launch("top-k select launch");
}

}  // namespace cs
