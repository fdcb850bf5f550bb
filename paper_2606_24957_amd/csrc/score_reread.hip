// score_reread.hip -- Eq. 5 with K read twice, for calls whose logits take more memory than K (33
// to 64 pairs over two KV heads of 64-element rows, such as every head of a draft layer: 56 pairs
// are 224 bytes of fp32 logits per position, written and read, against 256 bytes of K).
//
// The softmax of Eq. 5 needs each pair's max and sum over all N_b positions before any
// position's share is known.  Two kinds of workgroups, in one launch:
//   * first: per (layer, sequence, chunk of 512 or 1024 positions), the (max, sum of exp2) of every
//     column, stored write-through; the last chunk of a layer to count in merges them into
//     the columns' (M, 1 / Z).
//   * second: per (sequence, chunk), waits until the sequence's layers are merged, forms the
//     logits again from K and adds up sum_columns exp2(x - M) / Z over the layers.
// Bound by the reads of K: 24 layers of 16 x 32768 positions and 56 pairs (3.2 GB of K, 6.5 read from
// HBM) take 1.12 to 1.23 ms, 5.3 to 5.7 TB/s, against 1446 + 571 us with the logits written and read.
//
// The second kind's blocks of a unit (a sequence, or a (layer, sequence)) follow the first kind's of
// the unit `lag` later, so that they rarely wait.  The first kind waits for nothing, and on each XCD
// blocks are dispatched in id order, so that a launch of its own always goes on.  Beside another
// launch, second kinds of both may hold the slots of some XCD each that the other's first kind needs:
// a second-kind block waits for a bounded time only, and then forms the statistics of its unit
// itself, stores them where the first kind does (the same bits), and goes on.
#include "score_chunk.hpp"

namespace dustin {

namespace {

// counters of the sync region: chunks counted in per (layer, sequence); per sequence (or unit)
// merged layers (high half) and second-kind workgroups done (low half)
__device__ __forceinline__ int* first_count(const ChunkCall& a, int layer, int b) {
  return a.sync + (layer * a.batch + b) * a.sync_stride;
}
__device__ __forceinline__ int* second_count(const ChunkCall& a, int unit) {
  return a.sync + kScoreSyncMaxBatch + unit * a.sync_stride;
}
template <class S>
__device__ __forceinline__ float2* layer_stats(const ChunkCall& a, int layer, int b) {
  return reinterpret_cast<float2*>(a.stats) + ((int64_t)layer * a.batch + b) * (a.chunks + 1) * S::NC;
}

// The tw tiles (a multiple of four) of a layer, whose first three are in flight: every GS tiles,
// done(t0, x) gets the logits of tiles t0 .. t0 + GS - 1.  The three tiles from t_next on of the
// rows rs_next are in flight afterwards.
template <class S, class F>
__device__ __forceinline__ void stream_tiles(ScoreChunk<S>& k, __amdgpu_buffer_rsrc_t rs, int tw,
                                             __amdgpu_buffer_rsrc_t rs_next, int t_next, const u32x4 (&q)[S::CT][S::KS],
                                             F done) {
  static_assert(S::SPT == 1 && S::NB == 4, "a stage per tile");
  f32x4 x[S::GS][S::CT];
  for (int t = 0; t < tw; t += 4) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int tn = t + r + 3;
      k.issue(tn < tw ? rs : rs_next, tn < tw ? tn : t_next + tn - tw, 0, k.buf[(r + 3) % 4]);
      k.products(0, k.buf[r], q, x[r % S::GS]);
      __builtin_amdgcn_sched_barrier(0);  // tile by tile: hoisted loads would cost registers
      if (r % S::GS == S::GS - 1) done(t + r - (S::GS - 1), x);
    }
  }
}

// The (max, sum of exp2) of every column over chunk c of a layer, into the layer's statistics (by wave
// 0, complete when it goes on).
template <class S>
__device__ __forceinline__ void store_summary(const ChunkCall& a, int layer, int b, int c, ChunkLds& lds) {
  constexpr int CT = S::CT, GS = S::GS, NC = S::NC;
  static_assert(S::LB == 1 && NC <= kWave, "one lane per column");
  ScoreChunk<S> k(a, layer, b, c, lds);
  k.rows(a.tw);
  const auto rs = k.rsrc(layer);
#pragma unroll
  for (int r = 0; r < 3; ++r) k.issue(rs, r, 0, k.buf[r]);
  k.columns();
  u32x4 q[CT][S::KS];
  k.load_q(layer, q);
  k.sign_q(q);
  float m[1][CT], ssum[1][CT];
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) {
    m[0][ct] = -INFINITY;
    ssum[0][ct] = 0.f;
  }
  // (past the last tile, the chunk's last three again: in flight or in L2)
  stream_tiles(k, rs, a.tw, rs, a.tw - 3, q, [&](int t0, f32x4 (&x)[GS][CT]) {
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      const float mg = k.group_max(t0, ct, x);
      float add = 0.f;
#pragma unroll
      for (int i = 0; i < GS; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) add += k.weight(x[i][ct][e], mg);
      merge_ms(m[0][ct], ssum[0][ct], mg, add);
    }
  });
  k.summarise(m, ssum);
  __syncthreads();
  if (k.wave == 0) {
    if (k.lane < NC) {
      const float2 v = k.workgroup_summary(k.lane);
      store_pair_sc1(layer_stats<S>(a, layer, b) + c * NC + k.lane, v.x, v.y);
    }
    k.stores_done();
  }
}

// Adds to the unit's counter of merged layers (high half) and finished second-kind blocks (low half);
// whoever completes both returns it to zero.
__device__ __forceinline__ void count_second(const ChunkCall& a, int unit, int add, int G) {
  int* const ready = second_count(a, unit);
  const int all = (a.per_layer ? 1 : a.n_layers) << 16 | G;
  if (__hip_atomic_fetch_add(ready, add, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + add == all)
    __hip_atomic_store(ready, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A block of unit (layer0, b): of the first kind, chunk c of layer layer0 + l, or (l < 0) of the second
// kind, chunk c.
template <class S, bool kSum>
__device__ __forceinline__ void score_block(const ChunkCall& a, int layer0, int b, int l, int c, ChunkLds& lds) {
  constexpr int CT = S::CT, GS = S::GS, NC = S::NC, KS = S::KS;
  const bool first = l >= 0;
  ScoreChunk<S> k(a, layer0, b, c, lds);
  const int C = kChunkWaves * 16 * a.tw, G = (k.N + C - 1) / C;
  if (c >= G) return;  // uniform over the workgroup
  const int L = kSum ? a.n_layers : 1, unit = kSum ? b : layer0 * a.batch + b;
  if (!first) {
    k.rows(a.tw);
#pragma unroll
    for (int r = 0; r < 3; ++r) k.issue(k.rsrc(layer0), r, 0, k.buf[r]);
    if (threadIdx.x == 0) lds.go[0] = wait_count<16>(second_count(a, unit), 16, L, a.polls);
    asm volatile("" ::: "memory");  // the columns are read only after the count is complete
    __syncthreads();
  }
  if (first || !lds.go[0]) {  // the statistics of one chunk, or of all of the unit's
    const int l_end = first ? l + 1 : L, c_end = first ? c + 1 : G;
    for (l = first ? l : 0; l < l_end; ++l) {
      const int layer = layer0 + l;
      for (int cc = first ? c : 0; cc < c_end; ++cc) {
        store_summary<S>(a, layer, b, cc, lds);
        if (first && threadIdx.x == 0)
          lds.go[0] = __hip_atomic_fetch_add(first_count(a, layer, b), 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == G - 1;
        __syncthreads();
      }
      if (first && !lds.go[0]) return;
      k.place();
      float2* const stats = layer_stats<S>(a, layer, b);
      k.merge_chunks(stats, G, lds.mz + (first ? 0 : l * NC));
      if (first) {  // the last chunk of its layer
        if (k.wave == 0) {
          if (k.lane < NC) store_pair_sc1(stats + a.chunks * NC + k.lane, lds.mz[k.lane].x, lds.mz[k.lane].y);
          k.stores_done();
          if (k.lane == 0) {
            __hip_atomic_store(first_count(a, layer, b), 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            count_second(a, unit, 0x10000, G);
          }
        }
        return;
      }
    }
    k.place();
    k.rows(a.tw);
#pragma unroll
    for (int r = 0; r < 3; ++r) k.issue(k.rsrc(layer0), r, 0, k.buf[r]);
  }
  k.columns();
  u32x4 q[CT][KS];
  if (kSum) {  // every layer's queries as the lanes take them, by wave 0
    if (k.wave == 0)
      for (int l = 0; l < L; ++l) {
        u32x4 ql[CT][KS];
        k.load_q(layer0 + l, ql);
        k.sign_q(ql);
#pragma unroll
        for (int t = 0; t < CT; ++t)
#pragma unroll
          for (int kk = 0; kk < KS; ++kk) lds.q[((l * CT + t) * KS + kk) * kWave + k.lane] = ql[t][kk];
      }
  } else {
    k.load_q(layer0, q);
    k.sign_q(q);
  }
  if (lds.go[0]) {
    for (int i = threadIdx.x; i < L * NC; i += kChunkThreads)
      lds.mz[i] = load_pair_sc1(layer_stats<S>(a, layer0 + i / NC, b) + a.chunks * NC + i % NC);
  }
  __syncthreads();
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};  // lane lr: tile lr's positions 4 lg .. + 3
  for (int l = 0; l < L; ++l) {
    if (kSum) {
#pragma unroll
      for (int t = 0; t < CT; ++t)
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) q[t][kk] = lds.q[((l * CT + t) * KS + kk) * kWave + k.lane];
    }
    float2 mz[CT];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) mz[ct] = lds.mz[l * NC + ct * 16 + k.lr];
    // then the next layer's rows, or (past the last layer) the last three tiles again
    const bool more = l + 1 < L;
    stream_tiles(k, k.rsrc(layer0 + l), a.tw, k.rsrc(layer0 + (more ? l + 1 : l)), more ? 0 : a.tw - 3, q,
                 [&](int t0, f32x4 (&x)[GS][CT]) {
                   f32x4 y[GS];
#pragma unroll
                   for (int i = 0; i < GS; ++i) y[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                   for (int ct = 0; ct < CT; ++ct) {
                     if (!k.col_ok[ct]) continue;  // (it may hold anything: the caller's padding)
#pragma unroll
                     for (int i = 0; i < GS; ++i)
#pragma unroll
                       for (int e = 0; e < 4; ++e)
                         y[i][e] = fmaf(fast_exp2(fmaf(x[i][ct][e], k.scale, -mz[ct].x)), mz[ct].y, y[i][e]);
                   }
#pragma unroll
                   for (int i = 0; i < GS; ++i)
#pragma unroll
                     for (int e = 0; e < 4; ++e) {
                       const float w = sum_row16(y[i][e]);
                       acc[e] += k.lr == t0 + i ? w : 0.f;
                     }
                 });
  }
  if (a.hist) {
    __syncthreads();  // the queries have been read
    clear_hist(lds);
    __syncthreads();
  }
  k.write(acc, layer0, 0, a.tw);
  k.flush_hist();
  if (threadIdx.x == 0) count_second(a, unit, 1, G);
}

// Block order: `lag` units' first kind, then unit after unit the first kind of unit j and the second
// kind of unit j - lag, then the last `lag` units' second kind.  (No block is empty but past a
// sequence's end: blocks go to the XCDs and on to their shader engines in turn, so that a regular
// pattern of empty ones leaves some of them without work: 4 layers of 16 x 8192, 56 pairs, took 91 us.)
template <class S, bool kSum>
__global__ __launch_bounds__(kChunkThreads, 3) void score_reread_kernel(ChunkArgs args) {
  __shared__ __attribute__((aligned(16))) ChunkLds lds;
  const ChunkCall& a = args.call[0];
  const int layers = kSum ? a.n_layers : 1, firsts = layers * a.chunks, per = firsts + a.chunks;
  const int head = args.lag * firsts, body = (args.units - args.lag) * per;
  int id = blockIdx.x, u, r;  // unit; below firsts: its first kind
  if (id < head) {
    u = id / firsts;
    r = id - u * firsts;
  } else if ((id -= head) < body) {
    u = id / per;
    r = id - u * per;
    u += r < firsts ? args.lag : 0;
  } else {
    id -= body;
    u = id / a.chunks;
    r = firsts + id - u * a.chunks;
    u += args.units - args.lag;
  }
  const int part = u / a.batch, b = u - part * a.batch;  // the unit's layer (per-layer outputs), else 0
  const int l = r / a.chunks, c = r - l * a.chunks;
  score_block<S, kSum>(a, part, b, r < firsts ? l : -1, c, lds);
}

using Shape = ChunkShape<64, 2, 2, 4, 1, 2>;

}  // namespace

// Two column tiles for each of two KV heads of 64-element rows: 33 to 64 pairs, whose logits
// would be more bytes written and read than K is read again.
bool score_reread_supported(const ChunkCall& c) {
  return c.head_dim == 64 && c.nu == 2 && c.nt == 2 && (c.per_layer || c.n_layers * 4 <= kChunkMaxQ);
}

hipError_t launch_score_reread(const ChunkArgs& args, hipStream_t stream) {
  const ChunkCall& a = args.call[0];
  const bool sum = a.n_layers > 1 && !a.per_layer;
  const dim3 grid(args.units * ((sum ? a.n_layers : 1) + 1) * a.chunks), block(kChunkThreads);
  if (sum) hipLaunchKernelGGL((score_reread_kernel<Shape, true>), grid, block, 0, stream, args);
  else hipLaunchKernelGGL((score_reread_kernel<Shape, false>), grid, block, 0, stream, args);
  return hipGetLastError();
}

}  // namespace dustin
