// The decode and prefill planners, and utility kernels.
#include "kernels.h"

namespace tlf {

namespace {

// ---------------------------------------------------------------------------
// Decode planner: one workgroup of NT threads (the batch rounded up to whole
// waves, at most kPlanThreads), thread t owning sequences t, t + NT, ...
// Steps:
//   1. depth-sorted order, deepest first and stable in b, by a counting sort
//      whose ranks come from wave ballots: A_i = rows [0, n_i) (Eq. 4-6);
//   2. one new page for every executed (b, i) whose next slot starts a page,
//      numbered by a block prefix sum (deterministic);
//   3. statistics;
//   4. per executed (b, i): the slot's position, cache_len += 1, and the
//      slot's element offset for the QKV epilogue, by compact row.
// All global reads are issued at the start and all slot stores come last,
// after the final barrier (a barrier waits for outstanding stores).
// Dense mode (gather-scatter off): rows stay in batch order and every loop up
// to the deepest token of the step has all B rows; the rows of exited tokens
// get kv_slot -1 (no cache entry) and their attention reads the cache as it
// stands, which the statistics count.
// ---------------------------------------------------------------------------
constexpr int kPlanWaves = kPlanThreads / kWave;

// Running totals of the step statistics: an atomic add returns nothing to
// wait for, where a read-modify-write would cost a memory round trip.
__device__ __forceinline__ void add_stat(long long* p, unsigned long long v) {
  atomicAdd(reinterpret_cast<unsigned long long*>(p), v);
}
constexpr int kPlanChunks = 4;  // kPlanThreads * kPlanChunks >= max batch (NT = kPlanThreads above kPlanThreads sequences)

// NCH chunks of NT sequences, RL loops at most.
template <int NCH, int RL>
__global__ __launch_bounds__(kPlanThreads) void k_plan_decode(DecodePlanArgs a) {
  const CacheView& c = a.c;
  const int tid = threadIdx.x, lane = lane_id(), wv = tid >> 6, B = a.B, R = c.R;
  const int NT = blockDim.x, NW = NT / kWave;  // threads (a multiple of the wave) and waves
  __shared__ int cnt[kMaxLoops + 1];
  __shared__ int start[kMaxLoops + 1];
  __shared__ int fill[kMaxLoops + 1];
  __shared__ int wcnt[kPlanWaves][kMaxLoops + 1];
  __shared__ int scan_tmp[kPlanWaves + 1];
  __shared__ unsigned long long s_kvread;
  __shared__ int s_top, s_base;
  __shared__ int s_nact[kMaxLoops];

  // the global reads of the first NT sequences (every batch up to
  // that size) are issued here: depth, sequence length, the R cache lengths
  // and the allocator in one round trip, then the page-table entry of each
  // cache's partly filled last page; sequences beyond (chunks >= 1) read
  // theirs where they are used
  int m_of[NCH], row_of[NCH];
#pragma unroll
  for (int ch = 0; ch < NCH; ++ch) {
    const int b = ch * NT + tid;
    m_of[ch] = b < B ? a.depth[b] : 0;
    row_of[ch] = -1;
  }
  int seq0, len0[RL], page0[RL];
  {
    // clamped into range rather than guarded: a load under a lane's condition
    // can cost a round trip of its own.  Threads past the batch read its last
    // sequence and a loop past R the last loop; both have no depth to use it.
    const int b = max(0, min(tid, B - 1));
    seq0 = c.seq_len[b];
#pragma unroll
    for (int i = 0; i < RL; ++i) len0[i] = c.cache_len[b * R + min(i, R - 1)];
#pragma unroll
    for (int i = 0; i < RL; ++i)  // used where the depth runs loop i and its next slot starts no page
      page0[i] = c.page_table[((int64_t)b * R + min(i, R - 1)) * c.pages_per_seq +
                              min(len0[i] / kPage, c.pages_per_seq - 1)];
  }
  const int base0 = *c.page_next;
  auto len_at = [&](int ch, int b, int i) __attribute__((always_inline)) {
    return ch == 0 ? len0[i] : c.cache_len[b * R + i];
  };
  if (tid <= kMaxLoops) { cnt[tid] = 0; fill[tid] = 0; }
  if (tid == 0) { s_kvread = 0ull; s_base = base0; }
  __syncthreads();
#pragma unroll
  for (int ch = 0; ch < NCH; ++ch)
    if (m_of[ch] > 0) atomicAdd(&cnt[m_of[ch]], 1);
  __syncthreads();
  if (tid == 0) {
    int s = 0, top = 0;
    for (int m = R; m >= 1; --m) { start[m] = s; s += cnt[m]; if (top == 0 && cnt[m] > 0) top = m; }
    for (int i = 1; i <= R; ++i) {
      const int n = a.dense ? (i <= top ? B : 0) : start[i] + cnt[i];  // n_i = #{m >= i}
      a.nact[i - 1] = n;
      s_nact[i - 1] = n;
    }
    s_top = top;
  }
  __syncthreads();
  const int top = s_top;

  // 1. rank of b among the sequences of its depth with smaller b
  const unsigned long long below = (1ull << lane) - 1ull;
#pragma unroll
  for (int ch = 0; ch < NCH; ++ch) {
    if (ch * NT >= B) break;  // uniform
    const int m = m_of[ch];
    int rank = 0;
    for (int dv = 1; dv <= R; ++dv) {
      const unsigned long long mask = __ballot(m == dv);
      if (m == dv) rank = __popcll(mask & below);
      if (lane == 0) wcnt[wv][dv] = __popcll(mask);
    }
    __syncthreads();
    if (m > 0) {
      int off = 0;
      for (int w = 0; w < wv; ++w) off += wcnt[w][m];
      const int b = ch * NT + tid;
      const int row = a.dense ? b : start[m] + fill[m] + off + rank;
      row_of[ch] = row;
    }
    __syncthreads();
    if (tid >= 1 && tid <= R) {
      int t = 0;
      for (int w = 0; w < NW; ++w) t += wcnt[w][tid];
      fill[tid] += t;
    }
    __syncthreads();
  }

  // 2. pages needed: (b, i) for i < m_b whose next slot starts a page; each
  // row's first new page follows from a block prefix sum (every thread
  // carries the running total, so no barrier is needed between chunks), and
  // the entries each row's attention reads
  int ex_of[NCH];
  int total = 0;
  unsigned long long rd_sum = 0ull;
  const int lim_all = a.dense ? top : 0;  // dense: loops every row reads
#pragma unroll
  for (int ch = 0; ch < NCH; ++ch) {
    ex_of[ch] = 0;
    if (ch * NT >= B) break;  // uniform
    const int b = ch * NT + tid, m = m_of[ch];
    int need = 0;
    unsigned long long rd = 0ull;
#pragma unroll
    for (int i = 0; i < RL; ++i) {
      if (m > 0 && i < m) {
        const int len = len_at(ch, b, i);
        need += len % kPage == 0;
        rd += (unsigned long long)(len + 1);
      } else if (m > 0 && i < lim_all) {  // dense: computed and discarded
        rd += (unsigned long long)len_at(ch, b, i);
      }
    }
    rd_sum += rd;
    int tot;
    ex_of[ch] = total + block_exclusive_scan(need, scan_tmp, &tot);
    total += tot;
  }
  // one LDS atomic per wave (a same-address atomic from every lane serialises)
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) rd_sum += shfl_xor(rd_sum, o);
  if (lane == 0 && rd_sum != 0ull) atomicAdd(&s_kvread, rd_sum);
  const int base = s_base;
  const bool oom = (int64_t)base + total > c.max_pages;
  if (tid == 0 && oom) set_err(c.err, kErrOutOfPages);
  __syncthreads();

  // 3. bookkeeping, before any slot is written (a barrier after global
  // stores would wait for them): the depth histogram, the deepest depth and
  // the entries written follow from the per-depth counts
  if (tid == 0 && !oom) *c.page_next = base + total;
  if (tid < R) atomicAdd(&c.depth_hist[tid], (unsigned long long)cnt[tid + 1]);
  if (tid == 0) {
    unsigned long long kvw = 0ull;
    for (int dv = 1; dv <= R; ++dv) kvw += (unsigned long long)dv * cnt[dv];
    if (oom) kvw = 0ull;
    const unsigned long long kvr = oom ? 0ull : s_kvread;
    c.step_stats[kStatKvRead] = (long long)(kvr * (unsigned long long)a.kv_entry_bytes);
    c.step_stats[kStatKvWrite] = (long long)(kvw * (unsigned long long)a.kv_entry_bytes);
    c.step_stats[kStatLoops] = top;
    add_stat(c.step_stats + kStatStepsTotal, 1ull);
    add_stat(c.step_stats + kStatKvWriteTotal, kvw * (unsigned long long)a.kv_entry_bytes);
    add_stat(c.step_stats + kStatLoopsTotal, (unsigned long long)top);
    if (!oom) {
      // each executed (loop, layer) attention reads every valid entry of its
      // cache plus one q row and writes one o row per active token; summed
      // over layers: entry bytes times (entries read + active rows)
      unsigned long long rows = 0;
      for (int i = 0; i < R; ++i)
        rows += (unsigned long long)(a.dense ? (i < top ? B : 0) : start[i + 1] + cnt[i + 1]);
      add_stat(c.step_stats + kStatAttnBytesTotal, (kvr + rows) * (unsigned long long)a.kv_entry_bytes);
    }
  }
  if (tid < R) {
    if (oom) a.nact[tid] = 0;  // the step becomes a no-op: no active rows
    c.step_stats[kStatRows + tid] = oom ? 0 : s_nact[tid];
  }

  // 4. slots of the executed (b, i): positions, cache lengths, new pages and
  // each compact row's slot offset, and the row order; no barrier follows
  // these stores
#pragma unroll
  for (int ch = 0; ch < NCH; ++ch) {
    if (ch * NT >= B) break;  // uniform
    const int b = ch * NT + tid, m = m_of[ch];
    if (m > 0 && !oom) {
      int len[RL], page[RL];
      const int lim = a.dense ? top : m;  // loops whose cache this row reads
#pragma unroll
      for (int i = 0; i < RL; ++i) {
        len[i] = i < lim ? len_at(ch, b, i) : 0;
        page[i] = ch == 0 ? page0[i] : -1;
      }
      if (ch > 0) {
#pragma unroll
        for (int i = 0; i < RL; ++i)
          if (i < m && len[i] % kPage != 0)
            page[i] = c.page_table[((int64_t)b * R + i) * c.pages_per_seq + len[i] / kPage];
      }
      int next = base + ex_of[ch];
      const int t = ch == 0 ? seq0 : c.seq_len[b];
#pragma unroll
      for (int i = 0; i < RL; ++i) {
        if (i < m) {
          const int slot = len[i];
          if (slot % kPage == 0) {
            page[i] = next++;
            c.page_table[((int64_t)b * R + i) * c.pages_per_seq + slot / kPage] = page[i];
          }
          c.pos[(int64_t)page[i] * kPage + slot % kPage] = t;
          c.cache_len[b * R + i] = slot + 1;
          a.kv_slot[(int64_t)i * B + row_of[ch]] = (int64_t)page[i] * c.page_elems + slot % kPage;
        } else if (i < lim) {  // dense: computed and discarded
          a.kv_slot[(int64_t)i * B + row_of[ch]] = -1;
        }
      }
    }
    if (m > 0) {
      c.seq_len[b] = (ch == 0 ? seq0 : c.seq_len[b]) + 1;
      a.perm[row_of[ch]] = b;
      if (a.row_depth) a.row_depth[row_of[ch]] = m;
    }
  }
}

// ---------------------------------------------------------------------------
// Prefill planner, first launch: workgroup g counts sequence b0 + g's tokens
// per loop (those of depth >= i + 1) into seq_cnt[g][i] and takes the new pages
// of its caches, the first of each into row_off[g][i].  A loop whose pages do
// not fit the pool has no rows: its tokens keep the state of the loops that fit.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_plan_count(PrefillPlanArgs a) {
  const int tid = threadIdx.x, g = blockIdx.x, T = a.T, R = a.c.R;
  __shared__ int hist[kMaxLoops], s_np[kMaxLoops];
  __shared__ int s_base;
  const int bi = (a.b0 + g) * R + tid;
  const int old = a.append && tid < R ? a.c.cache_len[bi] : 0;
  if (tid < kMaxLoops) hist[tid] = 0;
  __syncthreads();
  const int32_t* depth = a.depth + (int64_t)g * T;
  for (int t0 = 0; t0 < T; t0 += 256 * 4) {
    int m[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) m[u] = depth[min(t0 + u * 256 + tid, T - 1)];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const bool in = t0 + u * 256 + tid < T;
      for (int i = 0; i < R; ++i) {
        const unsigned long long who = __ballot(in && m[u] == i + 1);
        if (lane_id() == 0 && who) atomicAdd(&hist[i], __popcll(who));
      }
    }
  }
  __syncthreads();
  int n = 0, np = 0;
  if (tid < R) {
    for (int i = tid; i < R; ++i) n += hist[i];
    np = (old + n + kPage - 1) / kPage - (old + kPage - 1) / kPage;  // pages to take
    s_np[tid] = np;
    atomicAdd(&a.c.depth_hist[tid], (unsigned long long)hist[tid]);
  }
  __syncthreads();
  if (tid == 0) {
    int all = 0;
    for (int i = 0; i < R; ++i) all += s_np[i];
    s_base = all > 0 ? atomicAdd(a.c.page_next, all) : 0;
    a.c.seq_len[a.b0 + g] = a.pos0 + T;
  }
  __syncthreads();
  if (tid < R) {
    int base = s_base;
    for (int i = 0; i < tid; ++i) base += s_np[i];
    if (np > 0 && (int64_t)base + np > a.c.max_pages) {
      set_err(a.c.err, kErrOutOfPages);
      n = 0;
    }
    a.seq_cnt[g * R + tid] = n;
    a.row_off[g * R + tid] = base;
  }
}

// ---------------------------------------------------------------------------
// Second launch: workgroup (g, i) gathers rho^(i) = sort(A_i) over sequence
// b0 + g's T tokens (Eq. 6) by a prefix sum over the flags m_t >= i, into the
// compact rows that follow the earlier sequences', and places those n entries
// in slots [n_old, n_old + n) of cache (b, i): n_old = 0 for a new batch, the
// current length when the call continues the caches (a later prompt chunk).
// The partly filled last page is used first, then the new pages that the first
// launch took; every new slot records its original position (Section 3.3
// address translation).  chunk_len[b][i] = n, and row_off[g][i] becomes the
// first of the n rows.
// ---------------------------------------------------------------------------
constexpr int kPrePlanThreads = 256, kPrePlanTokens = 4;

__global__ __launch_bounds__(kPrePlanThreads) void k_plan_prefill(PrefillPlanArgs a) {
  const CacheView& c = a.c;
  const int tid = threadIdx.x, T = a.T, R = c.R;
  const int g = blockIdx.x, i = blockIdx.y;
  const int b = a.b0 + g, bi = b * R + i;
  const int64_t GT = (int64_t)a.G * T;
  __shared__ int scan_tmp[kPrePlanThreads / kWave + 1];
  const int n = a.seq_cnt[g * R + i], base = a.row_off[g * R + i];
  const int old = a.append ? c.cache_len[bi] : 0;
  const int p_old = (old + kPage - 1) / kPage;           // pages already holding entries
  const int np = (old + n + kPage - 1) / kPage - p_old;  // new pages, base .. base + np - 1
  // rows of the earlier sequences
  int before = 0;
  for (int gg = tid; gg < g; gg += kPrePlanThreads) before += a.seq_cnt[gg * R + i];
  int off;
  block_exclusive_scan(before, scan_tmp, &off);
  int32_t* pt = c.page_table + (int64_t)bi * c.pages_per_seq;
  const int last_page = old % kPage != 0 ? pt[p_old - 1] : -1;
  int32_t* idx = a.tok_idx + (int64_t)i * GT + off;
  int64_t* ks = a.kv_slot + (int64_t)i * GT + off;
  const int32_t* depth = a.depth + (int64_t)g * T;
  int e0 = 0;
  for (int t0 = 0; n > 0 && t0 < T; t0 += kPrePlanThreads * kPrePlanTokens) {
    const int tb = t0 + tid * kPrePlanTokens;
    int f[kPrePlanTokens], cnt = 0, tot;
#pragma unroll
    for (int u = 0; u < kPrePlanTokens; ++u) {
      const int m = depth[min(tb + u, T - 1)];
      f[u] = tb + u < T && m > i;
      cnt += f[u];
    }
    int e = e0 + block_exclusive_scan(cnt, scan_tmp, &tot);
#pragma unroll
    for (int u = 0; u < kPrePlanTokens; ++u) {
      if (!f[u]) continue;
      const int s = old + e, pi = s / kPage;
      const int page = pi < p_old ? last_page : base + (pi - p_old);
      idx[e] = g * T + tb + u;
      ks[e] = (int64_t)page * c.page_elems + s % kPage;
      c.pos[(int64_t)page * kPage + s % kPage] = a.pos0 + tb + u;
      ++e;
    }
    e0 += tot;
  }
  for (int p = tid; p < np; p += kPrePlanThreads) pt[p_old + p] = base + p;
  // slots of the last new page past the last entry are marked empty
  const int s = old + n + tid;
  if (np > 0 && tid < kPage && s < (p_old + np) * kPage) c.pos[(int64_t)(base + np - 1) * kPage + s % kPage] = -1;
  if (tid == 0) {
    c.cache_len[bi] = old + n;
    c.chunk_len[bi] = n;
    a.row_off[g * R + i] = off;
    if (g == a.G - 1) a.nact[i] = off + n;
  }
}

__global__ void k_fill_i32(int32_t* p, int32_t v, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) p[i] = v;
}
__global__ void k_fill_u64(unsigned long long* p, unsigned long long v, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) p[i] = v;
}
// one wave per row: the largest of its group keys (value, then lowest id)
__global__ void k_argmax_finalize(const unsigned long long* keys, int groups, int32_t* next, int B) {
  const int b = blockIdx.x * (blockDim.x / kWave) + (int)(threadIdx.x / kWave), lane = lane_id();
  if (b >= B) return;
  unsigned long long key = 0ull;
  for (int gi = lane; gi < groups; gi += kWave) {
    const unsigned long long k = keys[(int64_t)b * groups + gi];
    key = k > key ? k : key;
  }
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const unsigned long long other = shfl_xor(key, o);
    key = other > key ? other : key;
  }
  if (lane == 0) next[b] = (int32_t)(0xFFFFFFFFu - (unsigned)(key & 0xFFFFFFFFull));
}

int fill_grid(int64_t n) {
  int64_t g = (n + 255) / 256;
  if (g > 4096) g = 4096;
  return g < 1 ? 1 : (int)g;
}

}  // namespace

hipError_t launch_plan_decode(const DecodePlanArgs& a, hipStream_t s) {
  if (a.B < 0 || a.B > kPlanThreads * kPlanChunks) return hipErrorInvalidValue;
  // fewer threads for a small batch: the planner's many barriers then wait
  // for fewer waves
  const int nt = std::min(kPlanThreads, std::max(kWave, (a.B + kWave - 1) / kWave * kWave));
  // one chunk and eight loops cover most steps: one workgroup runs its code
  // once, so the unrolled code that it does not fetch is time saved (with the
  // clamped loads, 1 sequence 10.1 -> 7.3 us, 64 sequences 12.6 -> 8.6)
  if (a.B > kPlanThreads)
    hipLaunchKernelGGL((k_plan_decode<kPlanChunks, kMaxLoops>), dim3(1), dim3(nt), 0, s, a);
  else if (a.c.R > 8)
    hipLaunchKernelGGL((k_plan_decode<1, kMaxLoops>), dim3(1), dim3(nt), 0, s, a);
  else
    hipLaunchKernelGGL((k_plan_decode<1, 8>), dim3(1), dim3(nt), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_plan_prefill(const PrefillPlanArgs& a, hipStream_t s) {
  if (a.G <= 0) return hipSuccess;
  if (!a.nact || !a.seq_cnt || !a.row_off) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_plan_count, dim3(a.G), dim3(256), 0, s, a);
  hipLaunchKernelGGL(k_plan_prefill, dim3(a.G, a.c.R), dim3(kPrePlanThreads), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_fill_i32(int32_t* p, int32_t v, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill_i32, dim3(fill_grid(n)), dim3(256), 0, s, p, v, n);
  return hipGetLastError();
}
hipError_t launch_fill_u64(unsigned long long* p, unsigned long long v, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill_u64, dim3(fill_grid(n)), dim3(256), 0, s, p, v, n);
  return hipGetLastError();
}
hipError_t launch_argmax_finalize(const unsigned long long* keys, int groups, int32_t* next, int B, hipStream_t s) {
  if (B <= 0) return hipSuccess;
  if (B <= 0 || groups <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_argmax_finalize, dim3((B + 3) / 4), dim3(4 * kWave), 0, s, keys, groups, next, B);
  return hipGetLastError();
}

}  // namespace tlf
