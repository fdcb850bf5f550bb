// kv.hip -- the steps on either side of verification (Sec. 3.2): the target KV of the T_b
// verification tokens is written into the cache at positions [N_b, N_b + T_b) before the
// verification attention reads it, and afterwards the accepted tokens are kept by moving
// N_b past them; the rejected rows stay beyond N_b, unseen, until the next step's window
// overwrites them.
#include "kernels.hpp"

namespace dustin {

constexpr int kKvThreads = 256;

// One 16-byte chunk per thread; a workgroup belongs to one cache (K or V) and one sequence, whose
// lengths are scalar loads that run beside the threads' (token, KV head, chunk) arithmetic.
// Bound by its launch and chain of loads (lengths, page, row): with the row found by 64-bit divisions,
// 3.9 to 4.8 us a launch for one sequence, 5 rows of 8 KV heads, about 0.5 us more than now.
__global__ __launch_bounds__(kKvThreads) void kv_append_kernel(KvAppendArgs a, uint32_t parts, int b0) {
  const bool is_v = blockIdx.x & 1;
  const uint32_t seq = (blockIdx.x >> 1) / parts, part = (blockIdx.x >> 1) - seq * parts;
  const int b = b0 + (int)seq;
  const int T = a.dims.nq(b), N = a.dims.len(b);
  const uint32_t cpr = (uint32_t)a.head_dim / 8, heads = (uint32_t)a.num_kv_heads;  // chunks per row
  const uint32_t i = part * kKvThreads + threadIdx.x;
  const uint32_t r = i / cpr, chunk = i - r * cpr;
  const uint32_t t = r / heads, h = r - t * heads;
  if (t >= (uint32_t)T) return;
  const int64_t pos = (int64_t)N + t;
  const KvView& c = is_v ? a.v : a.k;
  int64_t row;
  if (c.page_table) {
    const int64_t slot = pos >> c.page_shift;
    if (slot >= c.max_pages) return;  // no page for this position: nothing is written
    const int page = clampi(c.page_table[(int64_t)b * c.max_pages + slot], 0, c.num_pages - 1);
    row = (int64_t)page * c.stride_page + (pos & ((1 << c.page_shift) - 1)) * c.stride_n;
  } else {
    if (pos >= c.capacity) return;
    row = (int64_t)b * c.stride_b + pos * c.stride_n;
  }
  const uint16_t* src = (is_v ? a.v_new : a.k_new) + (int64_t)b * (is_v ? a.v_sb : a.k_sb) +
                        (int64_t)t * (is_v ? a.v_st : a.k_st) + (int64_t)h * (is_v ? a.v_sh : a.k_sh);
  uint16_t* dst = const_cast<uint16_t*>(c.data) + row + (int64_t)h * c.stride_h;
  *reinterpret_cast<u32x4*>(dst + 8 * chunk) = *reinterpret_cast<const u32x4*>(src + 8 * chunk);
}

hipError_t launch_kv_append(const KvAppendArgs& a, hipStream_t stream) {
  const int64_t chunks = (int64_t)a.dims.nq_max * a.num_kv_heads * (a.head_dim / 8);  // of one sequence
  if (a.batch == 0 || chunks == 0) return hipSuccess;
  const int64_t parts = (chunks + kKvThreads - 1) / kKvThreads;
  const int64_t most = ((INT64_C(1) << 32) / kKvThreads - 1) / (2 * parts);  // sequences: a grid has less than 2^32 threads
  if (most < 1) return hipErrorInvalidValue;
  for (int64_t b0 = 0; b0 < a.batch; b0 += most) {
    const int64_t n = a.batch - b0 < most ? a.batch - b0 : most;
    hipLaunchKernelGGL(kv_append_kernel, dim3((unsigned)(2 * n * parts)), dim3(kKvThreads), 0, stream, a,
                       (uint32_t)parts, (int)b0);
  }
  return hipGetLastError();
}

__global__ __launch_bounds__(kKvThreads) void kv_commit_kernel(int32_t* seq_lens, const int32_t* accepted,
                                                               const int32_t* n_query, int nq_max, int batch) {
  const int b = blockIdx.x * kKvThreads + threadIdx.x;
  if (b >= batch) return;
  const int T = n_query ? clampi(n_query[b], 0, nq_max) : nq_max;
  seq_lens[b] += clampi(accepted[b], 0, T);
}

hipError_t launch_kv_commit(int32_t* seq_lens, const int32_t* accepted, const int32_t* n_query, int nq_max,
                            int batch, hipStream_t stream) {
  if (batch == 0) return hipSuccess;
  hipLaunchKernelGGL(kv_commit_kernel, dim3((batch + kKvThreads - 1) / kKvThreads), dim3(kKvThreads), 0, stream,
                     seq_lens, accepted, n_query, nq_max, batch);
  return hipGetLastError();
}

}  // namespace dustin
