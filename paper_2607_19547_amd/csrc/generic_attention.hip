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
// FMAs reach).  A key tile costs D/2 + 16 ceil(D/32) matrix instructions of 64
// cycles per wavefront; the loads (16 + 16 ceil(D/32) instructions at D = 128)
// stay below a quarter of that time in the address units, and K/V need 1/8 of
// the L1 rate, so LDS staging would add barriers and save nothing.
//
// Measured (4,096 float32 tokens, 512 selected rows, 16 query heads, 2 KV heads,
// D = 128, scatter included): 167 us, 77 TFLOP/s, against 2,870 us for one
// wavefront per (row, head) with scalar FMAs, which it replaces at every
// geometry (bf16 D = 64: 107 against 960 us; D = 512: 772 against 4,288 us; 64
// tokens of D = 16: 13 against 17 us).  The error against float64 is 5.6e-7 to
// 9.8e-7 over eight inputs, against 7.5e-7 to 1.1e-6 (shorter sums).  The
// longest row tile sets the time when there are about as many workgroups as CUs
// (there 4,096 keys against 3,072 on average); splitting it further would need
// a workspace, which these calls do not take.
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
// Wavefronts per workgroup, at most: eight (two per SIMD, 256 registers each),
// four where the accumulators alone need most of that.
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
  constexpr int kWavesMax = gen_waves(NB);
  constexpr int kGroups = NB <= 2 ? 1 : NB <= 4 ? 2 : NB <= 8 ? 4 : 8;  // load groups per tile, for K and for V
  constexpr int kSteps = 4 * NB / kGroups;   // K chunks per lane and group (each lane half takes every other chunk)
  constexpr int kVRows = 16 / kGroups;       // V rows per lane and group
  constexpr int kQW = 32 * NB + 4;           // Q row stride in LDS (floats): four pad words spread the banks
  constexpr int kMinD = NB <= 4 ? 32 * (NB - 1) : NB <= 8 ? 32 * (NB - 2) : 256;  // D > kMinD
  constexpr int ES = sizeof(E);
  typedef GenLoad<E> Ld;
  typedef typename Ld::chunk chunk;
  typedef typename Ld::elem elem;
  __shared__ __attribute__((aligned(16))) float lds[kGenQ * kQW > kWavesMax * kGenQ * kGenBufW ? kGenQ * kQW : kWavesMax * kGenQ * kGenBufW];
  __shared__ float s_m[kWavesMax][kGenQ], s_l[kWavesMax][kGenQ];
  __shared__ int s_tok[kGenQ];
  // rows of a.q and of the results that the query vectors have (the 64-bit
  // divisions behind them once per vector; once per element they took 1.3 us of
  // a 168 us layer and about as much of the 64-token composition)
  __shared__ int64_t s_qrow[kGenQ], s_orow[kGenQ];
  const int nw = blockDim.x >> 6;
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
      s_tok[tid] = t >= a.cs1 && t < a.T ? t : -1;  // out-of-contract index: no output
      s_qrow[tid] = a.q_by_slot ? ((int64_t)blockIdx.z * a.Hq + h) * a.n_sel + m
                                : ((int64_t)layer * a.Hq + h) * a.n + (t - a.cs1);
      s_orow[tid] = ((int64_t)layer * a.Hq + h) * a.n_sel + m;
    }
    __syncthreads();
    for (int i = tid; i < kGenQ * 32 * NB; i += blockDim.x) {
      const int r = i / (32 * NB), d = i - r * (32 * NB);
      float v = 0.f;
      if (s_tok[r] >= 0 && d < D) v = gen_value(((const E*)a.q)[s_qrow[r] * D + d]);
      lds[r * kQW + d] = v;
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

    // merge the wavefronts' parts: weights from the overall max, then the
    // head dimension 32 elements at a time
    l_run = half_sum(l_run);
    if (hi == 0) {
      s_m[wave][q] = m_run;
      s_l[wave][q] = l_run;
    }
    __syncthreads();  // (also: every wavefront is done with Q in LDS)
    float M = -INFINITY, L = 0.f;
    for (int w = 0; w < nw; ++w) M = fmaxf(M, s_m[w][q]);
    // (a part without a weight is left out; one whose scores are NaN has a max of
    // -inf too, but a sum of NaN)
    for (int w = 0; w < nw; ++w) L += s_l[w][q] == 0.f ? 0.f : s_l[w][q] * expf(s_m[w][q] - M);
    const float f = (m_run == -INFINITY ? 0.f : expf(m_run - M)) / L;
    if (wave == 0 && hi == 0 && g_q >= 0 && a.lse) a.lse[s_orow[q]] = M + logf(L);
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      if (32 * j < D) {  // (uniform)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          lds[(wave * kGenQ + q) * kGenBufW + 8 * (r >> 2) + 4 * hi + (r & 3)] = o[j][r] * f;
        __syncthreads();
        for (int i = tid; i < kGenQ * 32; i += blockDim.x) {
          const int r = i >> 5, d = 32 * j + (i & 31);
          if (d < D && s_tok[r] >= 0) {
            float v = 0.f;
            for (int w = 0; w < nw; ++w) v += lds[(w * kGenQ + r) * kGenBufW + (i & 31)];
            gen_store((E*)a.out + s_orow[r] * D + d, v);
          }
        }
        __syncthreads();  // the buffer (and s_tok, s_m) is written again
      }
    }
  }
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
  else CS_LAUNCH(tr, (sel_attn_generic<E, 16, Rows>), grid, block, 0, s, a, rows);
}

template <typename Rows>
static void launch_generic(const Geo& g, const GenAttnArgs& a, const Rows& rows, int layers, hipStream_t s) {
  static_assert(sizeof(GenAttnArgs) + sizeof(Rows) <= 4096, "kernel arguments within 4 KB");
  // a wavefront for every key tile of the cache, up to the kernel's most
  const int most = gen_waves((g.D + 31) / 32);
  const int64_t key_tiles = (g.T + kGenKeys - 1) / kGenKeys;
  int waves = 1;
  while (waves < most && waves < key_tiles) waves *= 2;
  const dim3 grid((unsigned)std::min<int64_t>(a.n_tiles * g.Hkv, kGenGridX), 1, layers), block(64 * waves);
  TraceScope tr("sel_attn_generic", s);
  if (g.dtype == CS_BF16) launch_generic_e<uint16_t>(a, rows, grid, block, tr, s);
  else launch_generic_e<float>(a, rows, grid, block, tr, s);
}

cs_status launch_attention_generic(const Geo& g, const CacheView& cv, int lb, int le, const int32_t* sel,
                                   int64_t n_sel, const void* qf, bool q_by_slot, void* out, float* lse,
                                   hipStream_t s, bool check_only) {
  const int layers = le - lb;
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
