// Causal GQA attention of the selected rows (Eq. 1) for every geometry outside
// the bf16 / head_dim 128 kernels: float32 caches, any even head_dim <= 512,
// any group size; float32 arithmetic throughout.
//
// A workgroup takes one KV head and 32 query vectors (selected rows x the
// group's query heads, row-major), its wavefronts interleave the 32-key tiles
// up to the last row's token and merge their (O, max, sum) through LDS at the
// end.  Both products run on v_mfma_f32_32x32x2_f32:
//   S^T = K Q^T     lane l: key l % 32, four consecutive elements of the row at
//                   a time (one 16-byte load feeds four products), Q from LDS;
//   O^T += V^T P^T  the score registers are the B operand as they are: register
//                   r of a lane holds key 8(r/4) + 4(l/32) + r%4 of the tile, so
//                   lane l loads V of exactly that key, elements l%32 + 32j
//                   (coalesced, no LDS, no shuffles).
// K and V go from memory to registers, one group of loads ahead of the
// products (kGroups groups per tile and operand, at most 32 registers each).
//
// Bound: the float32 matrix rate (256 flop per clock and CU, twice what plain
// FMAs reach).  A key tile costs 32 NB matrix instructions of 64 cycles per
// wavefront, half of them per product, where NB is the instance's blocks of 32
// elements (1, 2, 3, 4, 6, 8, 10, 12 or 16: D rounds up to one of them); the
// loads (16 + 16 NB instructions at D = 128) stay below a quarter of that time in
// the address units, and K/V need 1/8 of the L1 rate, so LDS staging would add
// barriers and save nothing.  Above D = 192 the instances spill (about 120 to 140
// registers with 8 blocks, 240 with 10, 500 with 12, outside most of the
// products; 1,140 to 1,250 with 16, whose accumulators, O and a tile of S, are more
// than the 256 accumulation registers, so that every group of products moves
// some of them).
//
// Measured (4,096 float32 tokens, 512 selected rows, 16 query heads, 2 KV heads,
// D = 128, scatter included): 163 us, 79 TFLOP/s, against 2,870 us for one
// wavefront per (row, head) with scalar FMAs, which it replaces (but for the
// shortest caches, see sel_attn_row).  The same layer, calls replayed back to
// back: float32 D = 128 186 against 2,874 us; bf16 D = 64 120 against 1,448; float32
// D = 320 448 against 6,529 and D = 512 1,629 against 10,095; 96 tokens of D = 258 38
// against 66, 64 tokens of D = 16 (4 query heads) 8.7 against 18.7.  The error
// against float64 is 5.6e-7 to 9.8e-7 over eight inputs, against 7.5e-7 to 1.1e-6
// (shorter sums).  The longest row tile sets the time when there are about as
// many workgroups as CUs (there 4,096 keys against 3,072 on average); splitting
// it further would need a workspace, which these calls do not take.
#include <math.h>

#include <algorithm>

#include "cs_common.h"

namespace cs {

struct GenAttnArgs {
  const void* q;
  const int32_t* sel;
  void* out;
  float* lse;
  int64_t T, n, n_sel, n_tiles;  // n_tiles: tiles of 32 query vectors per KV head
  int cs1, Hq, Hkv, G, D, lb;
  int q_by_slot;
  float scale;
};

constexpr int kGenQ = 32;       // query vectors per workgroup
constexpr int kGenKeys = 32;    // keys per tile
// Wavefronts per workgroup: eight (two per SIMD, 256 registers each), four where
// the accumulators alone need most of that.  A short cache has fewer key tiles;
// its other wavefronts share the loading of Q and the writing of the results
// (32 tokens, float32 D = 128: 16 us with eight wavefronts, 27 to 32 with one).
constexpr int gen_waves(int nb) { return nb <= 4 ? 8 : 4; }
constexpr int kGenBufW = 33;    // row stride (floats) of the merge buffer
constexpr int64_t kGenGridX = 1 << 22;

// Buffer loads of a lane's elements: `chunk` is four consecutive elements of a
// row, `elem` one.  Offsets past the buffer's range read as zeros.
template <typename E>
struct GenLoad;
template <>
struct GenLoad<float> {
  typedef u32x4 chunk;
  typedef uint32_t elem;
  static __device__ __forceinline__ chunk load4(__amdgpu_buffer_rsrc_t r, int off) {
    return __builtin_bit_cast(chunk, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
  }
  // the same through two loads, for rows that end inside a chunk
  static __device__ __forceinline__ chunk load22(__amdgpu_buffer_rsrc_t r, int off) {
    const u32x2 a = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
    const u32x2 b = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(r, off + 8, 0, 0));
    return chunk{a[0], a[1], b[0], b[1]};
  }
  static __device__ __forceinline__ elem load1(__amdgpu_buffer_rsrc_t r, int off) {
    return __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0);
  }
  static __device__ __forceinline__ float get(const chunk& c, int e) { return __uint_as_float(c[e]); }
  static __device__ __forceinline__ float one(elem x) { return __uint_as_float(x); }
};
template <>
struct GenLoad<uint16_t> {
  typedef u32x2 chunk;
  typedef uint16_t elem;
  static __device__ __forceinline__ chunk load4(__amdgpu_buffer_rsrc_t r, int off) {
    return __builtin_bit_cast(chunk, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
  }
  static __device__ __forceinline__ chunk load22(__amdgpu_buffer_rsrc_t r, int off) {
    return chunk{__builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0), __builtin_amdgcn_raw_buffer_load_b32(r, off + 4, 0, 0)};
  }
  static __device__ __forceinline__ elem load1(__amdgpu_buffer_rsrc_t r, int off) {
    return __builtin_amdgcn_raw_buffer_load_b16(r, off, 0, 0);
  }
  static __device__ __forceinline__ float get(const chunk& c, int e) { return e & 1 ? bf16_hi(c[e >> 1]) : bf16_lo(c[e >> 1]); }
  static __device__ __forceinline__ float one(elem x) { return bf16_to_f32(x); }
};
__device__ __forceinline__ float gen_value(float x) { return x; }
__device__ __forceinline__ float gen_value(uint16_t x) { return bf16_to_f32(x); }
__device__ __forceinline__ void gen_store(float* p, float x) { *p = x; }
__device__ __forceinline__ void gen_store(uint16_t* p, float x) { *p = f32_to_bf16(x); }

__device__ __forceinline__ int64_t uniform64(int64_t x) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane((int)(uint32_t)x);
  return ((int64_t)__builtin_amdgcn_readfirstlane((int)(x >> 32)) << 32) | lo;
}
// A uniform value the compiler cannot relate to earlier ones, so that what is
// computed from it is not kept in registers across the loops around it.
__device__ __forceinline__ int fresh(int x) {
  x = __builtin_amdgcn_readfirstlane(x);
  asm volatile("" : "+s"(x));
  return x;
}
__device__ __forceinline__ float half_max(float x) { return fmaxf(x, __shfl_xor(x, 32)); }
__device__ __forceinline__ float half_sum(float x) { return x + __shfl_xor(x, 32); }

// The buffer of the rows from token kt on (uniform): offset 0 is row kt's
// first byte, the range ends with the rows (or with the tile, whichever is
// nearer), so keys past the cache read as zeros.  A paged tile may cross into
// the next chunks: `rest` goes through them.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t gen_rsrc(const char* p, int rows, int rb) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)p, 0, min(rows, kGenKeys) * rb, 0x00020000);
}
template <typename Rows>
struct GenTile;
template <>
struct GenTile<FlatRows> {
  __device__ __forceinline__ void init() {}
  __device__ __forceinline__ bool cross(const FlatRows&, int) { return false; }
  __device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const FlatRows& r, bool val, int64_t plane, int kt, int rb) const {
    return gen_rsrc((val ? r.v : r.k) + (plane * r.T + kt) * rb, (int)r.T - kt, rb);
  }
  template <typename F>
  __device__ __forceinline__ void rest(const FlatRows&, bool, int64_t, int, int, F) const {}
};
template <int CAP>
struct GenTile<PagedRowsT<CAP>> {
  int c;  // chunk of the last tile asked for; tiles come in ascending order within an item
  __device__ __forceinline__ void init() { c = 0; }
  __device__ __forceinline__ bool cross(const PagedRowsT<CAP>& r, int kt) {
    while (c + 1 < r.n && r.start[c + 1] <= kt) ++c;
    return c + 1 < r.n && r.start[c + 1] < kt + kGenKeys;
  }
  __device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const PagedRowsT<CAP>& r, bool val, int64_t plane, int kt, int rb) const {
    const int len = r.start[c + 1] - r.start[c], at = kt - r.start[c];
    return gen_rsrc((val ? r.v[c] : r.k[c]) + (plane * len + at) * rb, len - at, rb);
  }
  // f(buffer, tile row of its first row) for every further chunk with rows in the tile
  template <typename F>
  __device__ __forceinline__ void rest(const PagedRowsT<CAP>& r, bool val, int64_t plane, int kt, int rb, F f) const {
    for (int d = c + 1; d < r.n && r.start[d] < kt + kGenKeys; ++d) {
      const int len = r.start[d + 1] - r.start[d];
      f(gen_rsrc((val ? r.v[d] : r.k[d]) + plane * len * rb, len, rb), r.start[d] - kt);
    }
  }
};

// NB: 32-element blocks of the head dimension, D <= 32 NB.
template <typename E, int NB, typename Rows>
__global__ __launch_bounds__(64 * gen_waves(NB)) void sel_attn_generic(const GenAttnArgs a, const Rows rows) {
  constexpr int nw = gen_waves(NB), kThreads = 64 * nw;
  constexpr int kGroups = NB <= 2 ? 1 : NB <= 4 ? 2 : NB <= 8 ? 4 : 8;  // load groups per tile, for K and for V
  constexpr int kSteps = 4 * NB / kGroups;   // K chunks per lane and group (each lane half takes every other chunk)
  constexpr int kVRows = 16 / kGroups;       // V rows per lane and group
  constexpr int kQW = 32 * NB + 4;           // Q row stride in LDS (floats): four pad words spread the banks
  constexpr int kMinD = NB <= 4 ? 32 * (NB - 1) : NB <= 12 ? 32 * (NB - 2) : 384;  // D > kMinD
  constexpr int ES = sizeof(E);
  typedef GenLoad<E> Ld;
  typedef typename Ld::chunk chunk;
  typedef typename Ld::elem elem;
  constexpr int kLds = kGenQ * kQW > nw * kGenQ * kGenBufW ? kGenQ * kQW : nw * kGenQ * kGenBufW;
  __shared__ __attribute__((aligned(16))) float lds[kLds];  // Q, later the parts of the results
  __shared__ float s_m[nw][kGenQ], s_l[nw][kGenQ];
  __shared__ int s_tok[kGenQ];
  // rows of a.q and of the results that the query vectors have (the 64-bit
  // divisions behind them once per vector; once per element they took 1.3 us of
  // a 168 us layer and about as much of the 64-token composition)
  __shared__ int64_t s_qrow[kGenQ], s_orow[kGenQ];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int q = lane & 31, hi = lane >> 5;
  const int layer = a.lb + blockIdx.z;
  const int D = a.D, G = a.G, rb = D * ES;

  for (int64_t it = blockIdx.x; it < a.n_tiles * a.Hkv; it += gridDim.x) {
    // KV head fastest: with two or more heads, workgroups on one XCD then see
    // few of them; longest row tiles first
    // (the divisions run on the vector unit: their uniform results go back to scalar registers)
    const int64_t slot = uniform64(it / a.Hkv);
    const int kv = __builtin_amdgcn_readfirstlane((int)(it - slot * a.Hkv));
    const int64_t x0 = (a.n_tiles - 1 - slot) * kGenQ;  // first query vector of the tile
    const int64_t plane = (int64_t)layer * a.Hkv + kv;
    if (tid < kGenQ) {
      const int64_t m = (x0 + tid) / G;
      const int h = kv * G + (int)(x0 + tid - m * G);
      int t = -1;
      if (m < a.n_sel) t = a.sel[m];
      const bool ok = t >= a.cs1 && t < a.T;  // out-of-contract index: no output
      s_tok[tid] = ok ? t : -1;
      s_qrow[tid] = !ok ? 0  // (loaded, not used)
                    : a.q_by_slot ? ((int64_t)blockIdx.z * a.Hq + h) * a.n_sel + m
                                  : ((int64_t)layer * a.Hq + h) * a.n + (t - a.cs1);
      s_orow[tid] = ((int64_t)layer * a.Hq + h) * a.n_sel + m;
    }
    __syncthreads();
    // Q into LDS, up to eight loads in flight per thread (loaded one by one, 32
    // rows of 512 elements took 64 round trips, most of a short cache's time)
    constexpr int kQPer = kGenQ * 32 * NB / kThreads, kQBatch = kQPer < 8 ? kQPer : 8;
    static_assert(kQPer % kQBatch == 0, "whole batches");
    int tq = tid;  // (opaque: its indices are not kept for the results)
    asm volatile("" : "+v"(tq));
#pragma unroll 1
    for (int k0 = 0; k0 < kQPer; k0 += kQBatch) {
      E v[kQBatch];
#pragma unroll
      for (int k = 0; k < kQBatch; ++k) {
        const int i = tq + (k0 + k) * kThreads, r = i / (32 * NB), d = i - r * (32 * NB);
        v[k] = ((const E*)a.q)[s_qrow[r] * D + min(d, D - 1)];
      }
#pragma unroll
      for (int k = 0; k < kQBatch; ++k) {
        const int i = tq + (k0 + k) * kThreads, r = i / (32 * NB), d = i - r * (32 * NB);
        lds[r * kQW + d] = s_tok[r] >= 0 && d < D ? gen_value(v[k]) : 0.f;
      }
    }
    __syncthreads();
    const int g_q = s_tok[q];
    int g_min = g_q >= 0 ? g_q : 0x7fffffff, g_max = g_q;
#pragma unroll
    for (int o = 1; o < 32; o <<= 1) {
      g_min = min(g_min, __shfl_xor(g_min, o));
      g_max = max(g_max, __shfl_xor(g_max, o));
    }
    g_min = __builtin_amdgcn_readfirstlane(g_min);
    g_max = __builtin_amdgcn_readfirstlane(g_max);

    f32x16 o[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j) o[j] = f32x16{};
    float m_run = -INFINITY, l_run = 0.f;
    GenTile<Rows> tile;
    tile.init();
    chunk kb[2][kSteps];
    elem vb[2][kVRows][NB];
    const int koff = q * rb + 4 * hi * ES;   // this lane's key row, first chunk
    const int voff = 4 * hi * rb + q * ES;   // this lane's first V row, first element

    // Group g of the tile's K chunks: chunk 2(g kSteps + s) + hi of row q.
    // Chunks past D read the next row; their products are masked.
    auto load_k = [&](int kt, bool cross, int g, chunk* buf) {
      const __amdgpu_buffer_rsrc_t r = tile.rsrc(rows, false, plane, kt, rb);
      const int at = koff + 8 * ES * g * kSteps;
      if (D & 2) {
#pragma unroll
        for (int s = 0; s < kSteps; ++s) buf[s] = Ld::load22(r, at + 8 * ES * s);
      } else {
#pragma unroll
        for (int s = 0; s < kSteps; ++s) buf[s] = Ld::load4(r, at + 8 * ES * s);
      }
      if (cross)
        tile.rest(rows, false, plane, kt, rb, [&](__amdgpu_buffer_rsrc_t r2, int first) {
#pragma unroll
          for (int s = 0; s < kSteps; ++s)
            if (q >= first) buf[s] = Ld::load22(r2, at - first * rb + 8 * ES * s);
        });
    };
    // Group g of the tile's V rows: rows 8(r/4) + 4hi + r%4, elements q + 32j
    // (past D: the next row's, whose sums are not stored).
    auto load_v = [&](int kt, bool cross, int g, elem (*buf)[NB]) {
      const __amdgpu_buffer_rsrc_t rv = tile.rsrc(rows, true, plane, kt, rb);
      const int rbl = fresh(rb);
#pragma unroll
      for (int u = 0; u < kVRows; ++u) {
        const int r = g * kVRows + u, at = voff + (8 * (r >> 2) + (r & 3)) * rbl;
#pragma unroll
        for (int j = 0; j < NB; ++j) buf[u][j] = Ld::load1(rv, at + 32 * j * ES);
      }
      if (cross)
        tile.rest(rows, true, plane, kt, rb, [&](__amdgpu_buffer_rsrc_t r2, int first) {
#pragma unroll
          for (int u = 0; u < kVRows; ++u) {
            const int r = g * kVRows + u, row = 8 * (r >> 2) + (r & 3);
            if (row + 4 * hi >= first) {
#pragma unroll
              for (int j = 0; j < NB; ++j) buf[u][j] = Ld::load1(r2, voff + (row - first) * rbl + 32 * j * ES);
            }
          }
        });
    };

    int kt = wave * kGenKeys;
    const int stride = nw * kGenKeys;
    bool cross = false, dropped = false;
    if (kt <= g_max) {
      cross = tile.cross(rows, kt);
      load_k(kt, cross, 0, kb[0]);
    }
    for (; kt <= g_max; kt += stride) {
      f32x16 s = f32x16{};
#pragma unroll
      for (int g = 0; g < kGroups; ++g) {
        if (g + 1 < kGroups) load_k(kt, cross, g + 1, kb[(g + 1) & 1]);
        else load_v(kt, cross, 0, vb[0]);
        __builtin_amdgcn_sched_barrier(0);  // the next group's loads stay ahead of this group's products
#pragma unroll
        for (int u = 0; u < kSteps; ++u) {
          const int d0 = 8 * (g * kSteps + u);  // the step's elements d0 + 4hi .. d0 + 4hi + 3
          const f32x4 qv = *(const f32x4*)(lds + q * kQW + d0 + 4 * hi);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            float kx = Ld::get(kb[g & 1][u], e);
            if (d0 + 8 > kMinD) kx = d0 + 4 * hi + (e & 2) < D ? kx : 0.f;
            s = __builtin_amdgcn_mfma_f32_32x32x2f32(kx, qv[e], s, 0, 0, 0);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      // scores of query q: register r holds key kt + 8(r/4) + 4hi + r%4
      const bool diag = kt + kGenKeys - 1 > g_min;  // (uniform) some row ends inside the tile
      const int lim = g_q - kt - 4 * hi;            // last visible key, less 4hi
      float mt = -INFINITY;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        s[r] *= a.scale;
        if (diag && 8 * (r >> 2) + (r & 3) > lim) s[r] = -INFINITY;
        mt = fmaxf(mt, s[r]);
      }
      mt = half_max(mt);
      if (__ballot(mt > m_run)) {
        const float m_new = fmaxf(m_run, mt);
        const float alpha = m_run == -INFINITY ? 0.f : expf(m_run - m_new);
        l_run *= alpha;
#pragma unroll
        for (int j = 0; j < NB; ++j) o[j] *= alpha;
        m_run = m_new;
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        // a masked key has weight zero whatever the running max is
        s[r] = s[r] == -INFINITY ? 0.f : expf(s[r] - m_run);
        l_run += s[r];
      }
      const int kn = kt + stride;
      bool cross_n = false;
#pragma unroll
      for (int g = 0; g < kGroups; ++g) {
        if (g + 1 < kGroups) {
          load_v(kt, cross, g + 1, vb[(g + 1) & 1]);
        } else if (kn <= g_max) {
          cross_n = tile.cross(rows, kn);
          load_k(kn, cross_n, 0, kb[0]);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (diag) {
          // A value beyond a row's token must not reach that row even if it
          // is not finite (0 x inf = NaN): such values of keys that some row
          // of the tile does not see are left out here and added after the
          // loop to the rows that see them.
#pragma unroll
          for (int u = 0; u < kVRows; ++u) {
            const int r = g * kVRows + u;
            const bool all_see = kt + 8 * (r >> 2) + 4 * hi + (r & 3) <= g_min;
#pragma unroll
            for (int j = 0; j < NB; ++j) {
              const bool drop = !all_see && !(fabsf(Ld::one(vb[g & 1][u][j])) < INFINITY);
              vb[g & 1][u][j] = drop ? 0 : vb[g & 1][u][j];
              dropped |= drop;
            }
          }
        }
#pragma unroll
        for (int u = 0; u < kVRows; ++u)
#pragma unroll
          for (int j = 0; j < NB; ++j)
            o[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(Ld::one(vb[g & 1][u][j]), s[g * kVRows + u], o[j], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
      cross = cross_n;
    }
    if (__ballot(dropped)) {  // (rare) the values left out above, each with a positive weight
      const int De = fresh(D), rbe = De * ES;  // (nothing of this block is worth a register before it)
      int hie = 4 * hi;
      asm volatile("" : "+v"(hie));
      for (kt = wave * kGenKeys; kt <= g_max; kt += stride) {
        if (kt + kGenKeys - 1 <= g_min) continue;
        for (int key = max(kt, g_min + 1); key < min(kt + kGenKeys, (int)a.T); ++key) {
          const E* vr = (const E*)rows.row(true, plane, key, rbe);
#pragma unroll
          for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
              const float v = gen_value(vr[min(32 * j + 8 * (r >> 2) + hie + (r & 3), De - 1)]);
              o[j][r] += key <= g_q && !(fabsf(v) < INFINITY) ? v : 0.f;
            }
        }
      }
    }

    // merge the wavefronts' parts (of those that have a key tile): weights from
    // the overall max, then the head dimension 32 elements at a time
    const int nk = min(nw, g_max / kGenKeys + 1);
    l_run = half_sum(l_run);
    if (hi == 0) {
      s_m[wave][q] = m_run;
      s_l[wave][q] = l_run;
    }
    __syncthreads();  // (also: every wavefront is done with Q in LDS)
    float M = -INFINITY, L = 0.f;
    for (int w = 0; w < nk; ++w) M = fmaxf(M, s_m[w][q]);
    // (a part without a weight is left out; one whose scores are NaN has a max of
    // -inf too, but a sum of NaN)
    for (int w = 0; w < nk; ++w) L += s_l[w][q] == 0.f ? 0.f : s_l[w][q] * expf(s_m[w][q] - M);
    const float f = (m_run == -INFINITY ? 0.f : expf(m_run - M)) / L;
    if (wave == 0 && hi == 0 && g_q >= 0 && a.lse) a.lse[s_orow[q]] = M + logf(L);
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      if (32 * j < D) {  // (uniform)
        if (wave < nk) {  // (uniform)
#pragma unroll
          for (int r = 0; r < 16; ++r)
            lds[(wave * kGenQ + q) * kGenBufW + 8 * (r >> 2) + 4 * hi + (r & 3)] = o[j][r] * f;
        }
        __syncthreads();
        int tr = tid;
        asm volatile("" : "+v"(tr));
        for (int i = tr; i < kGenQ * 32; i += kThreads) {
          const int r = i >> 5, d = 32 * j + (i & 31);
          if (d < D && s_tok[r] >= 0) {
            float v = 0.f;
            for (int w = 0; w < nk; ++w) v += lds[(w * kGenQ + r) * kGenBufW + (i & 31)];
            gen_store((E*)a.out + s_orow[r] * D + d, v);
          }
        }
        __syncthreads();  // the buffer (and s_tok, s_m) is written again
      }
    }
  }
}

// Caches of one or two key tiles: one wavefront per (row, query head), a lane per
// key for the scores and per element for the sums.  The tile kernel would leave
// the work to one or two wavefronts, whose loads and products then follow one
// another, whatever the number of keys; here every row has its own, and the time
// grows with the keys.  Up to 24 keys for rows of at most 128 elements, 40 for
// 384, 64 beyond (where the tile kernel spills most).  Measured, one layer, a
// fifth of the rows, time over the tile kernel's at 20, 28, 40, 56 and 64 keys: D =
// 16: 0.98, 1.21, 1.35, 1.70, 1.91; D = 128: 0.85, 0.88, 1.21, 1.47, 1.60; D = 256:
// 0.67, 0.83, 0.97, 1.29, 1.37; D = 512: 0.45, 0.57, 0.72, 0.92, 1.02 (8 to 80 us a
// layer; with nine tenths of the rows the lines would lie at two thirds of these).
static bool one_row_kernel(int64_t T, int D) { return T <= (D <= 128 ? 24 : D <= 384 ? 40 : 64); }
template <typename E, typename Rows>
__global__ __launch_bounds__(64) void sel_attn_row(const GenAttnArgs a, const Rows rows) {
  __shared__ float qs[512], ps[64];
  const int64_t m = blockIdx.x;
  const int h = blockIdx.y, kv = h / a.G, layer = a.lb + blockIdx.z, lane = threadIdx.x;
  const int t = a.sel[m];
  if (t < a.cs1 || t >= a.T) return;  // out-of-contract index: no output
  const E* qp = (const E*)a.q + (a.q_by_slot ? ((int64_t)blockIdx.z * a.Hq + h) * a.n_sel + m
                                             : ((int64_t)layer * a.Hq + h) * a.n + (t - a.cs1)) * a.D;
  const int64_t plane = (int64_t)layer * a.Hkv + kv;
  const int rb = a.D * (int)sizeof(E);
  for (int d = lane; d < a.D; d += 64) qs[d] = gen_value(qp[d]);
  __syncthreads();
  float s = -INFINITY;  // (T <= 64: every key has a lane)
  if (lane <= t) {
    const E* kr = (const E*)rows.row(false, plane, lane, rb);
    float dot = 0.f;
    for (int d = 0; d < a.D; ++d) dot = fmaf(qs[d], gen_value(kr[d]), dot);
    s = dot * a.scale;
  }
  float top = s;
#pragma unroll
  for (int o = 32; o; o >>= 1) top = fmaxf(top, __shfl_xor(top, o));
  const float p = lane <= t ? expf(s - top) : 0.f;
  float sum = p;
#pragma unroll
  for (int o = 32; o; o >>= 1) sum += __shfl_xor(sum, o);
  ps[lane] = p;
  __syncthreads();
  float acc[8] = {};
  for (int j = 0; j <= t; ++j) {
    const float pj = ps[j];
    const E* vr = (const E*)rows.row(true, plane, j, rb);
#pragma unroll
    for (int x = 0; x < 8; ++x)
      if (lane + 64 * x < a.D) acc[x] = fmaf(pj, gen_value(vr[lane + 64 * x]), acc[x]);
  }
  const int64_t orow = ((int64_t)layer * a.Hq + h) * a.n_sel + m;
  const float inv = 1.f / sum;
#pragma unroll
  for (int x = 0; x < 8; ++x)
    if (lane + 64 * x < a.D) gen_store((E*)a.out + orow * a.D + lane + 64 * x, acc[x] * inv);
  if (a.lse && lane == 0) a.lse[orow] = top + logf(sum);
}

template <typename E, typename Rows>
static void launch_generic_e(const GenAttnArgs& a, const Rows& rows, dim3 grid, dim3 block, TraceScope& tr,
                             hipStream_t s) {
  const int nb = (a.D + 31) / 32;
  if (nb <= 1) CS_LAUNCH(tr, (sel_attn_generic<E, 1, Rows>), grid, block, 0, s, a, rows);
  else if (nb <= 2) CS_LAUNCH(tr, (sel_attn_generic<E, 2, Rows>), grid, block, 0, s, a, rows);
  else if (nb <= 3) CS_LAUNCH(tr, (sel_attn_generic<E, 3, Rows>), grid, block, 0, s, a, rows);
  else if (nb <= 4) CS_LAUNCH(tr, (sel_attn_generic<E, 4, Rows>), grid, block, 0, s, a, rows);
  else if (nb <= 6) CS_LAUNCH(tr, (sel_attn_generic<E, 6, Rows>), grid, block, 0, s, a, rows);
  else if (nb <= 8) CS_LAUNCH(tr, (sel_attn_generic<E, 8, Rows>), grid, block, 0, s, a, rows);
  else if (nb <= 10) CS_LAUNCH(tr, (sel_attn_generic<E, 10, Rows>), grid, block, 0, s, a, rows);
  else if (nb <= 12) CS_LAUNCH(tr, (sel_attn_generic<E, 12, Rows>), grid, block, 0, s, a, rows);
  else CS_LAUNCH(tr, (sel_attn_generic<E, 16, Rows>), grid, block, 0, s, a, rows);
}

template <typename Rows>
static void launch_generic(const Geo& g, const GenAttnArgs& a, const Rows& rows, int layers, hipStream_t s) {
  static_assert(sizeof(GenAttnArgs) + sizeof(Rows) <= 4096, "kernel arguments within 4 KB");
  if (one_row_kernel(g.T, g.D)) {
    TraceScope tr("sel_attn_row", s);
    const dim3 grid((unsigned)a.n_sel, g.Hq, layers);
    if (g.dtype == CS_BF16) CS_LAUNCH(tr, (sel_attn_row<uint16_t, Rows>), grid, dim3(64), 0, s, a, rows);
    else CS_LAUNCH(tr, (sel_attn_row<float, Rows>), grid, dim3(64), 0, s, a, rows);
    return;
  }
  const dim3 grid((unsigned)std::min<int64_t>(a.n_tiles * g.Hkv, kGenGridX), 1, layers), block(64 * gen_waves((g.D + 31) / 32));
  TraceScope tr("sel_attn_generic", s);
  if (g.dtype == CS_BF16) launch_generic_e<uint16_t>(a, rows, grid, block, tr, s);
  else launch_generic_e<float>(a, rows, grid, block, tr, s);
}

cs_status launch_attention_generic(const Geo& g, const CacheView& cv, int lb, int le, const int32_t* sel,
                                   int64_t n_sel, const void* qf, bool q_by_slot, void* out, float* lse,
                                   hipStream_t s, bool check_only) {
  const int layers = le - lb;
  // the launch of a wavefront per row; the tile kernel's workgroups (at most
  // kGenGridX x layers, of 512 threads at most) are within the limits where it is
  static_assert(kGenGridX * 512 < int64_t(1) << 32, "work-items along x");
  const cs_status st = check_grid(n_sel, g.Hq, layers, 64, "selective attention");
  if (st || check_only) return st;
  GenAttnArgs a;
  a.q = qf;
  a.q_by_slot = q_by_slot ? 1 : 0;
  a.sel = sel;
  a.out = out;
  a.lse = lse;
  a.T = g.T;
  a.n = g.n;
  a.n_sel = n_sel;
  a.n_tiles = (n_sel * g.G + kGenQ - 1) / kGenQ;
  a.cs1 = (int)g.cs1;
  a.Hq = g.Hq;
  a.Hkv = g.Hkv;
  a.G = g.G;
  a.D = g.D;
  a.lb = lb;
  a.scale = (float)(1.0 / sqrt((double)g.D));
  if (cv.paged) launch_generic(g, a, cv.pages<kMaxPages>(g), layers, s);
  else launch_generic(g, a, cv.flat(g), layers, s);
  return check_launch("generic attention launch");
}

}  // namespace cs
