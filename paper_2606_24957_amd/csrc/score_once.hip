// score_once.hip -- Eq. 5 in one pass for small calls: few workgroups, a latency chain.
//
// One workgroup per (sequence or (layer, sequence), chunk of 256 or 512 positions) keeps the logits of
// its chunk in registers (one layer, or a draft's three at once), so that only the softmax
// statistics travel:
//   * every four tiles a lane takes the max of its 16 logits of a column and replaces them by
//     exp2(x - max); the workgroup merges (max, sum) per column over lanes and waves, publishes
//     them with write-through stores, counts itself in on the unit's counter and waits until
//     all G chunks of the unit have;
//   * it merges the G summaries in a fixed order, and every position gets
//     sum_columns exp2(x - M) / Z, one multiply-add per logit.
// Bound by its chain of memory round trips (rows, publish, count, summaries), which is why the
// chunks are small (the rows stream over all CUs), the three draft layers share one publish and
// wait, and a step's two calls one launch.  16-wave workgroups of 512 positions that waited
// once per layer, in two launches, took 22 + 36 us for a step of 4 x 8192 positions over two
// target and three draft KV heads' layers, now 19 in one; one sequence of 32768 took 49, now 21.
//
// A wait ends without a cooperative launch: workgroups are dispatched in id order on each XCD, and a
// unit's chunks have consecutive ids, so that they hold slots or are next in line.  But workgroups of
// launches on other streams may hold those slots while they wait for this one's, some on one XCD
// and some on another.  So a workgroup waits for a bounded time only, and then depends on nobody:
// it forms every chunk's statistics itself, stores them where their owners do (the same bits), and
// goes on.  The last chunk of a unit to leave returns the unit's counters to zero.
#include "score_chunk.hpp"

namespace dustin {

namespace {

// Chunks times columns up to which every workgroup merges all summaries itself: four rounds of
// loads, beyond which they cost more than another hand-off while no workgroup waits for a slot (one
// sequence of 131072 positions, three layers, 24 pairs: 44.9 us, shared 37.7).  With several rounds
// of workgroups the hand-off's round trips under load cost more than the loads do (8 x 65536:
// 127 us, shared 153), and the host leaves share_merge unset.
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
// x = exp2(logit - the group's max) and that max (log2 domain, scaled).
template <bool kKeep, class S>
__device__ __forceinline__ void chunk_logits(ScoreChunk<S>& k, f32x4 (&x)[S::LB][S::TW][S::CT],
                                             float (&gm)[S::LB][S::TW / S::GS][S::CT]) {
  constexpr int LB = S::LB, CT = S::CT, GS = S::GS;
  k.begin();
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
  k.summarise(m, ssum);
}

// Chunk c of a unit.  False when the wait for the others ran out: then kAlone does it, and waits
// for nobody.
template <class S, bool kAlone>
__device__ __forceinline__ bool score_once_chunk(const ChunkCall& a, int unit, int c, ChunkLds& lds) {
  constexpr int NC = S::NC, LB = S::LB, CT = S::CT, GS = S::GS, TW = S::TW;
  const int layer0 = a.per_layer ? unit / a.batch : 0;
  ScoreChunk<S> k(a, layer0, a.per_layer ? unit - layer0 * a.batch : unit, c, lds);
  const int G = (k.N + S::C - 1) / S::C;  // chunks of this sequence
  if (c >= G) return true;  // uniform over the workgroup
  if (a.hist) clear_hist(lds);  // the barriers below order this before the counting
  int* const cnt = a.sync + unit * a.sync_stride;
  int* const done = a.sync + kScoreSyncMaxBatch + unit * a.sync_stride;
  float2* const stats = reinterpret_cast<float2*>(a.stats) + (int64_t)unit * (a.chunks + 1) * NC;
  f32x4 x[LB][TW][CT];
  float gm[LB][TW / GS][CT];
  if (kAlone)
    for (k.c = 0; k.c < G; ++k.c) {
      chunk_logits<false>(k, x, gm);
      __syncthreads();
      if (k.wave == 0) {
        for (int col = k.lane; col < NC; col += kWave) {
          const float2 v = k.workgroup_summary(col);
          store_pair_sc1(stats + k.c * NC + col, v.x, v.y);
        }
        k.stores_done();
      }
      __syncthreads();  // the summary is stored, and the waves' have been read
    }
  k.c = c;
  chunk_logits<true>(k, x, gm);
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
        lds.go[0] = wait_count<1>(cnt, 0, G, a.polls);
      }
      asm volatile("" ::: "memory");  // the summaries are read only after the count is complete
    }
  }
  __syncthreads();
  if (G > 1) {
    if (!kAlone && !lds.go[0]) return false;
    constexpr int kCols = NC <= 16 ? 16 : (NC <= 32 ? 32 : (NC <= 64 ? 64 : 128));
    if (G * kCols <= kMergeAll || !a.share_merge) k.merge_chunks(stats, G, lds.mz);
    else merge_shared(k, stats, G, done);
    // the last chunk of the unit to leave returns its counters to zero
    if (threadIdx.x == 0 && (__hip_atomic_fetch_add(done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & 0xffff) == G - 1) {
      __hip_atomic_store(cnt, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(done, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
  // exp2(x - M) / Z = exp2(x - m_group) times exp2(m_group - M) / Z, over the columns that count:
  // the others may hold anything (a query row past nq_b is the caller's padding)
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};  // lane lr: tile lr's positions 4 lg .. + 3
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
        acc[e] = k.lr == g * GS + i ? w : acc[e];
      }
  }
  k.write(acc, layer0, 0, TW);
  k.flush_hist();
  return true;
}

template <class S>
__device__ __forceinline__ void score_once(const ChunkCall& a, int unit, int c, ChunkLds& lds) {
  if (score_once_chunk<S, false>(a, unit, c, lds)) return;
  asm volatile("" : "+s"(unit), "+s"(c));  // as ScoreChunk::place()
  (void)score_once_chunk<S, true>(a, unit, c, lds);
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
hipError_t launch(const ChunkArgs& a, hipStream_t stream) {
  constexpr bool kTwo = !std::is_same<S1, NoShape>::value;
  const int per = a.call[0].chunks + (kTwo ? a.call[1].chunks : 0);
  hipLaunchKernelGGL((score_once_kernel<S0, S1>), dim3(a.units * per), dim3(kChunkThreads), 0, stream, a);
  return hipGetLastError();
}

bool three_layers(const ChunkCall& c) { return c.n_layers == 3 && !c.per_layer; }

// one layer, pairs of all KV heads in one column tile
template <int D, int NU>
hipError_t launch_shared(const ChunkArgs& a, hipStream_t stream) {
  return a.call[0].tw == 8 ? launch<ChunkShape<D, NU, 0, 8>, NoShape>(a, stream)
                           : launch<ChunkShape<D, NU, 0, 4>, NoShape>(a, stream);
}

template <int D>
hipError_t launch_nu(const ChunkArgs& a, hipStream_t stream) {
  switch (a.call[0].nu) {
    case 1: return launch_shared<D, 1>(a, stream);
    case 2: return launch_shared<D, 2>(a, stream);
    case 3: return launch_shared<D, 3>(a, stream);
    case 4: return launch_shared<D, 4>(a, stream);
    default: return hipErrorInvalidValue;
  }
}

// a draft's three layers
template <int NT>
hipError_t launch_draft(const ChunkArgs& a, hipStream_t stream) {
  return a.call[0].tw == 8 ? launch<ChunkShape<64, 2, NT, 8, 3>, NoShape>(a, stream)
                           : launch<ChunkShape<64, 2, NT, 4, 3>, NoShape>(a, stream);
}

template <int NU, int TW>
hipError_t launch_pair_tw(const ChunkArgs& a, hipStream_t stream) {
  return a.call[1].nt == 0 ? launch<ChunkShape<128, NU, 0, TW>, ChunkShape<64, 2, 0, TW, 3>>(a, stream)
                           : launch<ChunkShape<128, NU, 0, TW>, ChunkShape<64, 2, 1, TW, 3>>(a, stream);
}

template <int NU>
hipError_t launch_pair(const ChunkArgs& a, hipStream_t stream) {
  return a.call[0].tw == 8 ? launch_pair_tw<NU, 8>(a, stream) : launch_pair_tw<NU, 4>(a, stream);
}

}  // namespace

// One layer per output (or a draft's three, over two KV heads of 64-element rows); pairs in one
// column tile, or (such a draft) one or two for each KV head.
bool score_once_supported(const ChunkCall& c) {
  const bool draft = c.head_dim == 64 && c.nu == 2;
  if (c.nt > 0 && !draft) return false;
  return c.n_layers == 1 || c.per_layer || (draft && c.nt < 2 && three_layers(c));
}

// a target call (one layer, one column tile), then a draft call (three layers), as a
// verification step scores them
bool score_once_pair_supported(const ChunkCall& c0, const ChunkCall& c1) {
  return c0.tw == c1.tw && c0.head_dim == 128 && c0.nt == 0 && c0.n_layers == 1 &&
         (c0.nu == 1 || c0.nu == 2 || c0.nu == 4) && c1.head_dim == 64 && c1.nu == 2 && c1.nt <= 1 && three_layers(c1);
}

hipError_t launch_score_once(const ChunkArgs& a, int n_calls, hipStream_t stream) {
  const ChunkCall& c = a.call[0];
  if (n_calls == 2) switch (c.nu) {
      case 1: return launch_pair<1>(a, stream);
      case 2: return launch_pair<2>(a, stream);
      case 4: return launch_pair<4>(a, stream);
      default: return hipErrorInvalidValue;
    }
  if (three_layers(c)) return c.nt == 0 ? launch_draft<0>(a, stream) : launch_draft<1>(a, stream);
  if (c.nt == 0) return c.head_dim == 128 ? launch_nu<128>(a, stream) : launch_nu<64>(a, stream);
  return c.nt == 1 ? launch<ChunkShape<64, 2, 1, 4>, NoShape>(a, stream)
                   : launch<ChunkShape<64, 2, 2, 4>, NoShape>(a, stream);
}

}  // namespace dustin
