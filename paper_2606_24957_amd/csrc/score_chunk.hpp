// score_chunk.hpp -- what score_once.hpp and score_reread.hip share: a workgroup of four waves
// streams the K rows of a chunk of positions and forms the logits of Eq. 5's (head, query) pairs.
//
// Wave w takes TW tiles of 16 consecutive positions.  A tile's K rows meet the pairs' columns on
// MFMA 16x16x32.  NT = 0: one tile of 16 columns for the pairs of all NU KV heads (a column
// keeps its own head's products).  NT >= 1: NT column tiles for each KV head.  Lane (row r,
// group q) gets the logits of positions 4q .. 4q + 3 of the tile for column r of each column
// tile.  The rows stream through a ring of four 64-byte-per-lane register stages (three in
// flight while one is computed), through buffer loads at 32-bit offsets.
#pragma once

#include <type_traits>

#include "kernels.hpp"

// A call's outputs have the same bits alone and beside another call in one launch: no multiply
// and add is fused but where the code says so.
#pragma clang fp contract(off)

namespace dustin {

namespace {

constexpr int kChunkThreads = kChunkWaves * kWave;
constexpr int kChunkMaxCols = 96;     // columns of one publish: layers held at once times column tiles times 16
constexpr int kChunkMergeLoads = 8;   // summaries a thread loads at once when it merges

// (m, s) <- the union of two (max, sum of exp2(x - max)) summaries (score_sync.hip has its own, with
// the fusing left to the compiler)
__device__ __forceinline__ void merge_ms(float& m, float& s, float mo, float so) {
  const float mn = fmaxf(m, mo);
  const float mu = mn == -INFINITY ? 0.f : mn;
  s = fmaf(so, fast_exp2(mo - mu), s * fast_exp2(m - mu));
  m = mn;
}

// Sum over the 16 lanes of a row (rotations by 8, 4, 2, 1), the same in every lane.
template <int kCtrl>
__device__ __forceinline__ float add_ror(float x) {
  return x + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), kCtrl, 0xf, 0xf, true));
}
__device__ __forceinline__ float sum_row16(float x) {
  x = add_ror<0x128>(x);
  x = add_ror<0x124>(x);
  x = add_ror<0x122>(x);
  return add_ror<0x121>(x);
}

// LDS of a workgroup: byte offsets of the rows its waves read, the waves' and the slices'
// summaries, the columns' (M, 1 / Z), several layers' queries as the lanes take them, then the
// chunk's outputs by top key digit.
struct ChunkLds {
  uint32_t row[kChunkWaves * kChunkMaxTW * 16];
  float2 st[kChunkWaves][kChunkMaxCols];
  float2 part[kChunkThreads];
  float2 mz[kChunkMaxQ * 16];
  int go[2];  // the waits' outcomes, for the workgroup
  union {
    u32x4 q[kChunkMaxQ * 2 * kWave];
    uint32_t hist[kDigitBins];
  };
};

// Shapes: row length, used KV heads, column tiles per KV head (0: one tile shared by all),
// tiles per wave, layers held at once, tiles handed on together, and (score_once.hpp) whether LB layers
// follow LB layers.
template <int D_, int NU_, int NT_, int TW_, int LB_ = 1, int GS_ = 4, bool kLoop_ = false>
struct ChunkShape {
  static constexpr int D = D_, NU = NU_, NT = NT_, TW = TW_, LB = LB_;
  static constexpr bool kLoop = kLoop_;
  static constexpr int CT = NT == 0 ? 1 : NU * NT;  // column tiles
  static constexpr int KS = D / 32;                 // MFMA k-steps of one KV head's row
  static constexpr int HPS = 4 / KS;                // KV heads per load stage (64 bytes per lane)
  static constexpr int SPT = (NU + HPS - 1) / HPS;  // load stages per tile
  static constexpr int NST = TW * SPT;              // load stages per layer
  static constexpr int NS = LB * NST;               // load stages of the layers held at once
  static constexpr int NB = 4;                      // load stages in a ring: three in flight, one computed
  static constexpr int C = kChunkWaves * TW * 16;    // positions per workgroup
  static constexpr int NC = LB * CT * 16;           // columns of one publish
  static constexpr int GS = GS_;                    // tiles whose logits share a max
  static_assert(TW % GS == 0 && TW <= kChunkMaxTW && NC <= kChunkMaxCols && NS % NB == 0, "shape");
};
struct NoShape {};

// One workgroup's part of a call: chunk c of unit `unit`.
template <class S>
struct ScoreChunk {
  static constexpr int D = S::D, NU = S::NU, NT = S::NT, TW = S::TW, LB = S::LB, CT = S::CT, KS = S::KS,
                       HPS = S::HPS, SPT = S::SPT, NST = S::NST, NS = S::NS, NB = S::NB, C = S::C, NC = S::NC,
                       GS = S::GS;
  const ChunkCall& a;
  ChunkLds& lds;
  int c, b, layer0, lane, wave, lr, lg, N, nq, p0, cu;
  bool col_ok[CT];
  int64_t q_off[CT], k_off;
  uint32_t* my_row;
  uint32_t sh, flip, keep;
  float scale;
  u32x4 buf[NB][4];
  u32x4 bq[LB][CT][KS];

  __device__ __forceinline__ ScoreChunk(const ChunkCall& a_, int layer0_, int b_, int c_, ChunkLds& lds_)
      : a(a_), lds(lds_), c(c_), b(b_), layer0(layer0_) {
    place();
    N = a.dims.len(b);
  }

  // This thread's place, opaque to the compiler: a second pass over chunks (after a wait that ran
  // out) would otherwise share what the first one computed from it, in registers held all the while.
  __device__ __forceinline__ void place() {
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    lane = t & (kWave - 1);
    wave = __builtin_amdgcn_readfirstlane(t / kWave);
    lr = lane & 15;
    lg = lane >> 4;
  }

  // Row offsets, the first load stages of the layers from layer0 on, columns and queries.
  __device__ __forceinline__ void begin() {
    place();
    rows(TW);
    first_stages();
    columns();
    queries();
  }
  __device__ __forceinline__ void first_stages() {
#pragma unroll
    for (int qi = 0; qi < NB - 1; ++qi) issue(rsrc(layer0 + qi / NST), qi % NST / SPT, qi % SPT, buf[qi]);
  }
  __device__ __forceinline__ void queries() {
#pragma unroll
    for (int lb = 0; lb < LB; ++lb) load_q(layer0 + lb, bq[lb]);
  }

  // Byte offsets of the rows of this wave's tw tiles (clamped to the last position; paged rows
  // through the page table), kept in LDS so that a stage's loads wait for no other load.
  __device__ __forceinline__ void rows(int tw) {
    p0 = (c * kChunkWaves + wave) * tw * 16;  // this wave's first position
    my_row = lds.row + wave * tw * 16;
    const uint32_t sn = (uint32_t)a.k.stride_n * 2u;
    for (int i = 0; i < tw * 16; i += kWave) {
      const int p = min(p0 + i + lane, N - 1);
      uint32_t off;
      if (a.k.page_table) {
        const int page =
            clampi(a.k.page_table[(int64_t)b * a.k.max_pages + (p >> a.k.page_shift)], 0, a.k.num_pages - 1);
        off = (uint32_t)page * ((uint32_t)a.k.stride_page * 2u) + (uint32_t)(p & ((1 << a.k.page_shift) - 1)) * sn;
      } else {
        off = (uint32_t)p * sn;
      }
      my_row[i + lane] = off;
    }
    sh = (uint32_t)a.k.stride_h * 2u;
    k_off = a.k.page_table ? 0 : (int64_t)b * a.k.stride_b;
  }

  // Column lr of column tile t: (query head, query) on used KV head cu (NT = 0).  A column past
  // the pairs, or of a query past nq_b, repeats the tile's first column and is left out of the
  // sums (col_ok): with nq_b = 0, or an empty tile, that one may itself hold anything.
  __device__ __forceinline__ void columns() {
    nq = a.dims.nq(b);
    cu = 0;
#pragma unroll
    for (int t = 0; t < CT; ++t) {
      const bool in = lr < a.cols[t] && (int)a.col_query[t * 16 + lr] < nq;
      const int col = t * 16 + (in ? lr : 0);
      col_ok[t] = in;
      if (NT == 0) cu = a.col_u[col];
      q_off[t] = (int64_t)b * a.q_sb + (int64_t)a.col_query[col] * a.q_sj + (int64_t)a.col_head[col] * a.q_sh + 8 * lg;
    }
    // The logits are scaled by a positive number: a negative scale flips the queries' signs,
    // and a scale of zero clears them.
    flip = a.scale_log2 < 0.f ? 0x80008000u : 0u;
    keep = a.scale_log2 == 0.f ? 0u : ~0u;
    scale = a.scale_log2 == 0.f ? 1.f : fabsf(a.scale_log2);
  }

  __device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(int l) const {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(a.k_layers[l] + k_off), 0, a.extent, 0x00020000);
  }
  // stage s of tile t: KV heads s HPS .. s HPS + HPS - 1, in the MFMA A layout (row lr,
  // elements 32 kk + 8 lg .. + 7)
  __device__ __forceinline__ void issue(__amdgpu_buffer_rsrc_t rs, int t, int s, u32x4 (&dst)[4]) const {
    const uint32_t off = my_row[t * 16 + lr] + 16u * lg;
#pragma unroll
    for (int h = 0; h < HPS; ++h) {
      const int u = s * HPS + h;
      if (u < NU) {
#pragma unroll
        for (int kk = 0; kk < KS; ++kk)
          dst[h * KS + kk] = __builtin_bit_cast(
              u32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, off, (int)((uint32_t)a.kv[u] * sh + 64u * kk), 0));
      }
    }
  }
  // B operands of layer l: column lr's query, elements 32 kk + 8 lg .. + 7
  __device__ __forceinline__ void load_q(int l, u32x4 (&dst)[CT][KS]) const {
#pragma unroll
    for (int t = 0; t < CT; ++t)
#pragma unroll
      for (int kk = 0; kk < KS; ++kk) dst[t][kk] = load16(a.q_layers[l] + q_off[t] + 32 * kk);
  }
  __device__ __forceinline__ void sign_q(u32x4 (&q)[CT][KS]) const {  // see columns()
    if (flip == 0u && keep != 0u) return;
#pragma unroll
    for (int t = 0; t < CT; ++t)
#pragma unroll
      for (int kk = 0; kk < KS; ++kk) q[t][kk] = (q[t][kk] & keep) ^ flip;
  }

  // Stage s's products with layer q's columns into the logits x of its tile (unscaled).
  __device__ __forceinline__ void products(int s, const u32x4 (&k)[4], const u32x4 (&q)[CT][KS], f32x4 (&x)[CT]) const {
#pragma unroll
    for (int h = 0; h < HPS; ++h) {
      const int u = s * HPS + h;
      if (u < NU) {
        constexpr int kTiles = NT == 0 ? 1 : NT;
#pragma unroll
        for (int j = 0; j < kTiles; ++j) {
          const int ct = NT == 0 ? 0 : u * NT + j;
          f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int kk = 0; kk < KS; ++kk) v = mfma16x16x32(as_bf16x8(k[h * KS + kk]), as_bf16x8(q[ct][kk]), v);
          if (NT == 0 && u > 0) {
#pragma unroll
            for (int e = 0; e < 4; ++e) x[0][e] = cu == u ? v[e] : x[0][e];
          } else {
            x[ct] = v;
          }
        }
      }
    }
  }

  // The logits of the layers from l0 on that are held at once, whose first stages are in
  // flight: every GS tiles, done(lb, g, x) gets those of group g (x[i][ct]: tile g GS + i).
  template <class F>
  __device__ __forceinline__ void stream(int l0, F done) {
    __amdgpu_buffer_rsrc_t rs[LB];
#pragma unroll
    for (int lb = 0; lb < LB; ++lb) rs[lb] = rsrc(l0 + lb);
#pragma unroll
    for (int lb = 0; lb < LB; ++lb) sign_q(bq[lb]);
    f32x4 x[GS][CT];
#pragma unroll
    for (int qi = 0; qi < NS; ++qi) {
      const int lb = qi / NST, t = qi % NST / SPT, i = t % GS, s = qi % SPT, qn = qi + NB - 1;
      if (qn < NS) issue(rs[qn / NST], qn % NST / SPT, qn % SPT, buf[qn % NB]);
      products(s, buf[qi % NB], bq[lb], x[i]);
      __builtin_amdgcn_sched_barrier(0);  // stage by stage: hoisted loads would cost registers
      if (s == SPT - 1 && i == GS - 1) done(lb, t - (GS - 1), x);
    }
  }

  // A group's maximum of column tile ct (log2 domain, scaled), with the logits past N set to
  // -inf.
  __device__ __forceinline__ float group_max(int t0, int ct, f32x4 (&x)[GS][CT]) const {
    const int pg = p0 + t0 * 16;  // the group's first position
    if (pg + GS * 16 > N) {           // uniform
      int lim = N - pg - 4 * lg;
      asm volatile("" : "+v"(lim));  // keeps the compares here, out of scalar registers
#pragma unroll
      for (int i = 0; i < GS; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) x[i][ct][e] = 16 * i + e < lim ? x[i][ct][e] : -INFINITY;
    }
    float mx = -INFINITY;
#pragma unroll
    for (int i = 0; i < GS; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) mx = fmaxf(mx, x[i][ct][e]);
    return mx == -INFINITY ? -INFINITY : mx * scale;
  }
  __device__ __forceinline__ float weight(float x, float mg) const {  // exp2(logit - the group's max)
    return fast_exp2(fmaf(x, scale, mg == -INFINITY ? 0.f : -mg));
  }

  // The wave's (max, sum) of every column into LDS.
  __device__ __forceinline__ void summarise(float (&m)[LB][CT], float (&ssum)[LB][CT]) const {
#pragma unroll
    for (int lb = 0; lb < LB; ++lb)
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {
#pragma unroll
        for (int off = 16; off <= 32; off <<= 1) {
          const float mo = __shfl_xor(m[lb][ct], off), so = __shfl_xor(ssum[lb][ct], off);
          merge_ms(m[lb][ct], ssum[lb][ct], mo, so);
        }
        if (lg == 0) lds.st[wave][(lb * CT + ct) * 16 + lr] = make_float2(m[lb][ct], ssum[lb][ct]);
      }
  }
  // The workgroup's summary of column col, the waves merged in order.
  __device__ __forceinline__ float2 workgroup_summary(int col) const {
    float M = -INFINITY, Z = 0.f;
#pragma unroll
    for (int w = 0; w < kChunkWaves; ++w) merge_ms(M, Z, lds.st[w][col].x, lds.st[w][col].y);
    return make_float2(M, Z);
  }
  static __device__ __forceinline__ float2 normaliser(float M, float Z) {
    return make_float2(M == -INFINITY ? 0.f : M, Z > 0.f ? 1.f / Z : 0.f);
  }
  // All threads: the G chunks' summaries of a unit ([chunk][NC] at `stats`), slice sl merging
  // chunks sl, sl + kSlices, ... in order, then the slices in order: columns' (M, 1 / Z) into
  // mz (LDS).
  __device__ __forceinline__ void merge_chunks(const float2* stats, int G, float2* mz) const {
    constexpr int kCols = NC <= 16 ? 16 : (NC <= 32 ? 32 : (NC <= 64 ? 64 : 128));
    constexpr int kSlices = kChunkThreads / kCols;
    const int col = threadIdx.x % kCols, sl = threadIdx.x / kCols;
    if (col < NC) {
      float M = -INFINITY, Z = 0.f;
      for (int c0 = sl; c0 < G; c0 += kChunkMergeLoads * kSlices) {
        float2 v[kChunkMergeLoads];
#pragma unroll
        for (int i = 0; i < kChunkMergeLoads; ++i)
          v[i] = load_pair_sc1(stats + min(c0 + i * kSlices, G - 1) * NC + col);
#pragma unroll
        for (int i = 0; i < kChunkMergeLoads; ++i)
          if (c0 + i * kSlices < G) merge_ms(M, Z, v[i].x, v[i].y);
      }
      lds.part[sl * kCols + col] = make_float2(M, Z);
    }
    __syncthreads();
    if ((int)threadIdx.x < NC) {
      float M = -INFINITY, Z = 0.f;
#pragma unroll
      for (int i = 0; i < kSlices; ++i) {
        const float2 v = lds.part[i * kCols + threadIdx.x];
        merge_ms(M, Z, v.x, v.y);
      }
      mz[threadIdx.x] = normaliser(M, Z);
    }
    __syncthreads();
  }

  static __device__ __forceinline__ void stores_done() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): the write-through stores have completed
    asm volatile("" ::: "memory");
  }

  // out = init + acc for positions 4 lg .. + 3 of tile t0 + lr (lr < nt) below N_b, counted into
  // lds.hist
  __device__ __forceinline__ void write(const f32x4& acc, int l, int t0, int nt) const {
    const float* const init_row = a.init ? a.init + (int64_t)b * a.init_sb : nullptr;
    float* const out_row = a.out + (int64_t)b * a.out_sb + (a.per_layer ? (int64_t)l * a.out_sl : 0);
    const int n0 = p0 + (t0 + lr) * 16 + 4 * lg;
    if (lr >= nt || n0 >= N) return;
    f32x4 val;
    if (n0 + 3 < N && ((uintptr_t)(out_row + n0) & 15) == 0 && (!init_row || ((uintptr_t)(init_row + n0) & 15) == 0)) {
      const f32x4 in = init_row ? *reinterpret_cast<const f32x4*>(init_row + n0) : f32x4{0.f, 0.f, 0.f, 0.f};
      val = in + acc;
      *reinterpret_cast<f32x4*>(out_row + n0) = val;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        val[e] = (init_row && n0 + e < N ? init_row[n0 + e] : 0.f) + acc[e];
        if (n0 + e < N) out_row[n0 + e] = val[e];
      }
    }
    if (a.hist) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (n0 + e < N) atomicAdd(&lds.hist[order_key(val[e]) >> 20], 1u);
    }
  }

  // The chunk's outputs counted by top key digit: the non-zero bins go into the sequence's
  // histogram.
  __device__ __forceinline__ void flush_hist() const {
    if (!a.hist) return;
    __syncthreads();
    uint32_t* const gh = a.hist + (int64_t)b * kDigitBins;
    for (int i = threadIdx.x; i < kDigitBins; i += kChunkThreads) {
      const uint32_t v = lds.hist[i];
      if (v) __hip_atomic_fetch_add(gh + i, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
};

__device__ __forceinline__ void clear_hist(ChunkLds& lds) {
  for (int i = threadIdx.x; i < kDigitBins; i += kChunkThreads) lds.hist[i] = 0u;
}

// One lane waits until *word >> shift reaches `target`, for at most `polls` more looks at it.
template <int kSleep>
__device__ __forceinline__ bool wait_count(const int* word, int shift, int target, int polls) {
  for (; __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >> shift < target; --polls) {
    if (polls <= 0) return false;
    __builtin_amdgcn_s_sleep(kSleep);
  }
  return true;
}

}  // namespace

}  // namespace dustin
