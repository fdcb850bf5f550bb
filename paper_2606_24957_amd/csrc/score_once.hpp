// score_once.hpp -- Eq. 5 in one pass for small calls: few workgroups, a latency chain.
//
// One workgroup per (sequence or (layer, sequence), chunk of 256 or 512 positions) keeps the logits of
// its chunk in registers (one layer, or a draft's two, three or four at once; of more, one or two
// after the other), so that only the softmax statistics travel:
//   * every four tiles a lane takes the max of its 16 logits of a column and replaces them by
//     exp2(x - max); the workgroup merges (max, sum) per column over lanes and waves, publishes
//     them with write-through stores, counts itself in on the unit's counter and waits until
//     all G chunks of the unit have;
//   * it merges the G summaries in a fixed order, and every position gets
//     sum_columns exp2(x - M) / Z, one multiply-add per logit.
// Bound by its chain of memory round trips (rows, publish, count, summaries), which is why the
// chunks are small (the rows stream over all CUs), up to four draft layers share one publish and
// wait, and a step's two calls one launch.  16-wave workgroups of 512 positions that waited
// once per layer, in two launches, took 55 us for a step's scores of 4 x 8192 positions, over two
// KV heads of the target and three draft layers, now 15 in one; one sequence of 32768 took 73, now 19.
//
// A wait ends without a cooperative launch: workgroups are dispatched in id order on each XCD, and a
// unit's chunks have consecutive ids, so that they hold slots or are next in line.  But workgroups of
// launches on other streams may hold those slots while they wait for this one's, some on one XCD
// and some on another.  So a workgroup waits for a bounded time only, and then depends on nobody:
// it forms every chunk's statistics itself, stores them where their owners do (the same bits), and
// goes on.  The last chunk of a unit to leave returns the unit's counters to zero.
#pragma once

#include "score_chunk.hpp"

namespace dustin {

hipError_t launch_score_once_pair(const ChunkArgs& a, hipStream_t stream);  // score_once_pair.hip

namespace {

// Chunks times columns up to which every workgroup merges all summaries itself: four rounds of
// loads, beyond which they cost more than another hand-off while no workgroup waits for a slot (one
// sequence of 131072 positions, three layers, 24 pairs: 41.7 us, shared 38.3).  With several rounds
// of workgroups the hand-off's round trips under load cost more than the loads do (8 x 65536:
// 116 us, shared 123), and the host leaves share_merge unset.
constexpr int kMergeAll = 4 * kChunkThreads * kChunkMergeLoads;

// Column col's (M, 1 / Z) over the unit's G chunks, by one wave (lane 0 holds it).
template <class S>
__device__ __forceinline__ float2 merge_column(const ScoreChunk<S>& k, const float2* stats, int G, int col) {
  float M = -INFINITY, Z = 0.f;
  float2 v[kChunkMaxOnce / kWave];
#pragma unroll
  for (int i = 0; i < kChunkMaxOnce / kWave; ++i)
    v[i] = load_pair_sc1(stats + min(k.lane + i * kWave, G - 1) * S::NC + col);
#pragma unroll
  for (int i = 0; i < kChunkMaxOnce / kWave; ++i)
    if (k.lane + i * kWave < G) merge_ms(M, Z, v[i].x, v[i].y);
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const float mo = __shfl_xor(M, off), so = __shfl_xor(Z, off);
    merge_ms(M, Z, mo, so);
  }
  return k.normaliser(M, Z);
}

// The unit's workgroups share the merge of its G chunks' summaries: wave w of chunk c merges column
// c + w G and publishes its (M, 1 / Z) behind the summaries, counted in the high half of *done;
// every workgroup then reads all of them into lds.mz, or, should they not come, merges them all.
template <class S>
__device__ __forceinline__ void merge_shared(const ScoreChunk<S>& k, float2* stats, int G, int* done) {
  constexpr int NC = S::NC;
  const int col = k.c + k.wave * G;
  if (col < NC) {  // uniform over the wave
    const float2 n = merge_column(k, stats, G, col);
    if (k.lane == 0) store_pair_sc1(stats + k.a.chunks * NC + col, n.x, n.y);
    k.stores_done();
    if (k.lane == 0) __hip_atomic_fetch_add(done, 0x10000, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (threadIdx.x == 0) k.lds.go[1] = wait_count<1>(done, 16, NC, k.a.polls);
  asm volatile("" ::: "memory");  // the columns are read only after the count is complete
  __syncthreads();
  if (k.lds.go[1]) {
    if ((int)threadIdx.x < NC) k.lds.mz[threadIdx.x] = load_pair_sc1(stats + k.a.chunks * NC + threadIdx.x);
  } else {
    k.stores_done();  // this wave's count, before the workgroup's departure
    for (int t = k.wave; t < NC; t += kChunkWaves) {
      const float2 n = merge_column(k, stats, G, t);
      if (k.lane == 0) k.lds.mz[t] = n;
    }
  }
  __syncthreads();
}

// A wave's (max, sum of exp2) of every column over its chunk, into LDS.  With kKeep, also
// x = exp2(logit - the group's max) and that max (log2 domain, scaled).  `next`: rounds to come.
template <bool kKeep, class S>
__device__ __forceinline__ void chunk_logits(ScoreChunk<S>& k, f32x4 (&x)[S::LB][S::TW][S::CT],
                                             float (&gm)[S::LB][S::TW / S::GS][S::CT], int next) {
  constexpr int LB = S::LB, CT = S::CT, GS = S::GS;
  float m[LB][CT], ssum[LB][CT];
#pragma unroll
  for (int lb = 0; lb < LB; ++lb)
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      m[lb][ct] = -INFINITY;
      ssum[lb][ct] = 0.f;
    }
  k.stream(k.layer0, [&](int lb, int t0, f32x4 (&xg)[GS][CT]) {
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      const float mg = k.group_max(t0, ct, xg);
      float add = 0.f;
#pragma unroll
      for (int i = 0; i < GS; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float w = k.weight(xg[i][ct][e], mg);
          if (kKeep) x[lb][t0 + i][ct][e] = w;
          add += w;
        }
      if (kKeep) gm[lb][t0 / GS][ct] = mg;
      merge_ms(m[lb][ct], ssum[lb][ct], mg, add);
    }
  });
  if (S::kLoop && kKeep && next > 0) {  // the next layers' first rows and queries, across the wait
    k.layer0 += LB;
    k.first_stages();
    k.queries();
  }
  k.summarise(m, ssum);
}

// Chunk c of a unit.  The round whose wait for the others ran out, or -1: kAlone does it over, and
// waits for nobody (the workgroup has counted itself in up to round `counted`).
template <class S, bool kAlone>
__device__ __forceinline__ int score_once_chunk(const ChunkCall& a, int unit, int c, int counted, ChunkLds& lds) {
  constexpr int NC = S::NC, LB = S::LB, CT = S::CT, GS = S::GS, TW = S::TW;
  const int layer0 = a.per_layer ? unit / a.batch : 0;
  ScoreChunk<S> k(a, layer0, a.per_layer ? unit - layer0 * a.batch : unit, c, lds);
  const int G = (k.N + S::C - 1) / S::C;  // chunks of this sequence
  if (c >= G) return -1;  // uniform over the workgroup
  if (a.hist) clear_hist(lds);  // the barriers below order this before the counting
  int* const cnt = a.sync + unit * a.sync_stride;
  int* const done = a.sync + kScoreSyncMaxBatch + unit * a.sync_stride;
  const int rounds = S::kLoop ? a.n_layers / LB : 1;  // LB layers after LB layers
  float2* stats = reinterpret_cast<float2*>(a.stats) + (int64_t)unit * rounds * (a.chunks + 1) * NC;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};  // lane lr: tile lr's positions 4 lg .. + 3
  if (!kAlone) k.begin();
  for (int r = 0; r < rounds; ++r, stats += (a.chunks + 1) * NC) {
    f32x4 x[LB][TW][CT];
    float gm[LB][TW / GS][CT];
    if (kAlone) {
      k.layer0 = layer0 + r * LB;
      for (k.c = 0; k.c < G; ++k.c) {
        k.begin();
        chunk_logits<false>(k, x, gm, 0);
        __syncthreads();
        if (k.wave == 0) {
          for (int col = k.lane; col < NC; col += kWave) {
            const float2 v = k.workgroup_summary(col);
            store_pair_sc1(stats + k.c * NC + col, v.x, v.y);
          }
          k.stores_done();
          if (r > counted && k.c == c && k.lane == 0)
            __hip_atomic_fetch_add(cnt, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        __syncthreads();  // the summary is stored, and the waves' have been read
      }
      k.c = c;
      k.begin();
    }
    chunk_logits<true>(k, x, gm, kAlone ? 0 : rounds - 1 - r);
    __syncthreads();
    if (!kAlone && k.wave == 0) {  // publishes and waits
      for (int col = k.lane; col < NC; col += kWave) {
        const float2 v = k.workgroup_summary(col);
        if (G == 1) lds.mz[col] = k.normaliser(v.x, v.y);
        else store_pair_sc1(stats + c * NC + col, v.x, v.y);
      }
      if (G > 1) {
        k.stores_done();
        if (k.lane == 0) {
          __hip_atomic_fetch_add(cnt, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          lds.go[0] = wait_count<1>(cnt, 0, (r + 1) * G, a.polls);
        }
        asm volatile("" ::: "memory");  // the summaries are read only after the count is complete
      }
    }
    __syncthreads();
    if (G > 1) {
      if (!kAlone && !lds.go[0]) return r;
      constexpr int kCols = NC <= 16 ? 16 : (NC <= 32 ? 32 : (NC <= 64 ? 64 : 128));
      constexpr bool kNever = kChunkMaxOnce * kCols <= kMergeAll;
      static_assert(kNever || !S::kLoop, "a shared merge counts one round");
      if (kNever || G * kCols <= kMergeAll || !a.share_merge) k.merge_chunks(stats, G, lds.mz);
      else merge_shared(k, stats, G, done);
    }
    // exp2(x - M) / Z = exp2(x - m_group) times exp2(m_group - M) / Z, over the columns that count:
    // the others may hold anything (a query row past nq_b is the caller's padding)
#pragma unroll
    for (int g = 0; g < TW / GS; ++g) {
      f32x4 y[GS];
#pragma unroll
      for (int i = 0; i < GS; ++i) y[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {
        if (!k.col_ok[ct]) continue;
#pragma unroll
        for (int lb = 0; lb < LB; ++lb) {
          const float2 mz = lds.mz[(lb * CT + ct) * 16 + k.lr];
          const float mg = gm[lb][g][ct];
          // (the group that holds the maximum has factor 1 also where that is infinite)
          const float f = (mg == mz.x ? 1.f : fast_exp2(mg - mz.x)) * mz.y;
#pragma unroll
          for (int i = 0; i < GS; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) y[i][e] = fmaf(x[lb][g * GS + i][ct][e], f, y[i][e]);
        }
      }
#pragma unroll
      for (int i = 0; i < GS; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float w = sum_row16(y[i][e]);
          acc[e] = k.lr == g * GS + i ? (S::kLoop ? acc[e] + w : w) : acc[e];
        }
    }
  }
  // the last chunk of the unit to leave returns its counters to zero
  if (G > 1 && threadIdx.x == 0 &&
      (__hip_atomic_fetch_add(done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & 0xffff) == G - 1) {
    __hip_atomic_store(cnt, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(done, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  k.write(acc, layer0, 0, TW);
  k.flush_hist();
  return -1;
}

template <class S>
__device__ __forceinline__ void score_once(const ChunkCall& a, int unit, int c, ChunkLds& lds) {
  const int r = score_once_chunk<S, false>(a, unit, c, -1, lds);
  if (r < 0) return;
  asm volatile("" : "+s"(unit), "+s"(c));  // as ScoreChunk::place()
  (void)score_once_chunk<S, true>(a, unit, c, r, lds);
}

// The calls' chunks unit by unit: the first call's chunks of a unit, then the second's.
template <class S0, class S1>
__global__ __launch_bounds__(kChunkThreads, 2) void score_once_kernel(ChunkArgs a) {
  __shared__ __attribute__((aligned(16))) ChunkLds lds;
  constexpr bool kTwo = !std::is_same<S1, NoShape>::value;
  const int per = a.call[0].chunks + (kTwo ? a.call[1].chunks : 0);
  const int unit = blockIdx.x / per;
  const int c = blockIdx.x - unit * per;
  const int units0 = a.call[0].batch * (a.call[0].per_layer ? a.call[0].n_layers : 1);
  if (!kTwo || c < a.call[0].chunks) {
    if (unit < units0) score_once<S0>(a.call[0], unit, c, lds);
  } else if constexpr (kTwo) {
    if (unit < a.call[1].batch) score_once<S1>(a.call[1], unit, c - a.call[0].chunks, lds);
  }
}

template <class S0, class S1>
hipError_t launch_once(const ChunkArgs& a, hipStream_t stream) {
  constexpr bool kTwo = !std::is_same<S1, NoShape>::value;
  const int per = a.call[0].chunks + (kTwo ? a.call[1].chunks : 0);
  hipLaunchKernelGGL((score_once_kernel<S0, S1>), dim3(a.units * per), dim3(kChunkThreads), 0, stream, a);
  return hipGetLastError();
}

// The shape of a draft call (two KV heads of 64-element rows): up to four layers at once, of more two or
// one after the other; of 17 to 32 pairs three at once.
template <int TW, class F>
hipError_t draft_shape(const ChunkCall& c, F launch) {
  if (c.nt == 1) return launch(ChunkShape<64, 2, 1, TW, 3>());
  switch (c.n_layers) {
    case 1: return launch(ChunkShape<64, 2, 0, TW, 1>());
    case 2: return launch(ChunkShape<64, 2, 0, TW, 2>());
    case 3: return launch(ChunkShape<64, 2, 0, TW, 3>());
    case 4: return launch(ChunkShape<64, 2, 0, TW, 4>());
    default:
      return c.n_layers % 2 ? launch(ChunkShape<64, 2, 0, TW, 1, 4, true>()) : launch(ChunkShape<64, 2, 0, TW, 2, 4, true>());
  }
}

}  // namespace

}  // namespace dustin
