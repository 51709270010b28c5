// Ordered placement of a batch of decisions, every chain position of every
// placed request in parallel (ps_commit and the per-arrival scheduler's
// batches).
//
// What has to come out is what applying the entries one after the other
// gives: entry e's hit is measured against its instance's table as the
// entries before it left it, its new blocks join the instance's row in
// chain order until the cap, and every position refused past the cap counts.
// An entry-by-entry kernel (one wave per instance, 64 positions a step, each
// step waiting for its probes and inserts) took 25 ms for 512 requests of
// about 2,300 blocks on 64 instances: a serial chain of up to 16,000
// dependent steps on the busiest instance.  But the order only decides which
// occurrence of a block is its first one:
//   * positions are numbered in entry order inside each instance's group,
//     and the first occurrence of a block absent from the table is the least
//     number that carries it (atomicMin in a scratch set of the group);
//   * a block is present for entry e when the table has it or its first
//     occurrence lies before e, so e's hit is the least position without;
//   * the first occurrences, counted in order, are the row positions of the
//     new blocks, and the cap refuses exactly those whose rank reaches the
//     room left.
// Kernels: clear (scratch set), probe (table lookups, scratch set), mark (hits,
// first occurrences counted per chunk), scan (those counts), group (ranks at the
// group bounds), insert (table, row), drop (refused positions, where a cap
// binds) and state (counters; the scheduler's batches move them themselves).
// All but scan and group are bound by random 64-byte reads and memory-side
// atomics, so each thread keeps kCommitU positions in flight.

#include "ps_common.h"

namespace {

constexpr uint32_t kPosOld = 0xFFFFFFFFu;   // the table has the block
constexpr uint32_t kPosZero = 0xFFFFFFFEu;  // zero hash: never present, never inserted

constexpr int kCommitThreads = 256;
constexpr int kCommitU = 4;  // positions per thread and chunk
constexpr uint32_t kCommitChunk = kCommitThreads * kCommitU;
static_assert(kCommitChunk == kCommitChunkPositions, "chunk size shared with the host");
constexpr int kOffLds = 256;  // entry offsets of a chunk kept in LDS

// Last index e in [lo, hi) with off[e] <= p, given off[lo] <= p.
__device__ __forceinline__ uint32_t last_le(const uint32_t* off, uint32_t lo, uint32_t hi, uint32_t p) {
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) >> 1;
    if (off[mid] <= p) lo = mid;
    else hi = mid;
  }
  return lo;
}

// Entries of the chunk that starts at p0: the first one, and the offsets
// after it in LDS (all of the chunk's when it has at most kOffLds of them).
// Every thread of the workgroup calls it; ends with a barrier.
struct ChunkEntries {
  uint32_t e0, n;  // first entry; entries whose offsets are in LDS
};

__device__ __forceinline__ ChunkEntries chunk_entries(const CommitBatch& b, uint32_t n_ent,
                                                      uint32_t p0, uint32_t* lds) {
  ChunkEntries c;
  c.e0 = last_le(b.ent_off, 0u, n_ent, p0);
  c.n = n_ent - c.e0 < (uint32_t)kOffLds ? n_ent - c.e0 : (uint32_t)kOffLds;
  __syncthreads();  // the previous chunk's readers
  for (uint32_t k = threadIdx.x; k < c.n; k += blockDim.x) lds[k] = b.ent_off[c.e0 + k];
  __syncthreads();
  return c;
}

__device__ __forceinline__ uint32_t entry_of(const CommitBatch& b, uint32_t n_ent, const ChunkEntries& c,
                                             const uint32_t* lds, uint32_t p) {
  const uint32_t k = last_le(lds, 0u, c.n, p);
  // the last offset in LDS may not be the last entry at or before p
  if (k + 1 == c.n && c.e0 + c.n < n_ent) return last_le(b.ent_off, c.e0 + k, n_ent, p);
  return c.e0 + k;
}

// Scratch slot of `key` in the group's set (2 slots per position of the
// group), claimed if new.
__device__ __forceinline__ uint32_t set_claim(unsigned long long* keys, uint32_t base, uint32_t size,
                                              uint64_t key) {
  const uint32_t h = (uint32_t)((key * 0x9E3779B97F4A7C15ull) >> 32);
  uint32_t at = (uint32_t)(((uint64_t)h * size) >> 32);
  for (uint32_t step = 0; step < size; ++step) {
    // a stale read can only show an empty slot as empty: the swap decides
    unsigned long long v = keys[(size_t)base + at];
    if (v == 0ull) {
      v = atomicCAS(&keys[(size_t)base + at], 0ull, (unsigned long long)key);
      if (v == 0ull) return base + at;
    }
    if (v == (unsigned long long)key) return base + at;
    if (++at == size) at = 0u;
  }
  return base;  // not reached: the set has twice as many slots as positions
}

__global__ __launch_bounds__(kCommitThreads) void commit_clear_kernel(CommitBatch b) {
  const CommitHdr h = *b.hdr;
  const size_t slots = 2 * (size_t)h.n_pos;
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  const size_t t0 = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  for (size_t k = t0; k < slots; k += stride) b.set_key[k] = 0ull;
  for (size_t k = t0; k < slots; k += stride) b.set_pos[k] = 0xFFFFFFFFu;
  for (size_t e = t0; e < h.n_ent; e += stride) b.ent_hit[e] = b.ent_off[e + 1] - b.ent_off[e];
  if (t0 == 0) *b.cap_binds = 0u;
}

__global__ __launch_bounds__(kCommitThreads) void commit_probe_kernel(CommitBatch b) {
  __shared__ uint32_t lds[kOffLds];
  const CommitHdr h = *b.hdr;
  const uint32_t chunks = (h.n_pos + kCommitChunk - 1) / kCommitChunk;
  for (uint32_t ch = blockIdx.x; ch < chunks; ch += gridDim.x) {
    const uint32_t p0 = ch * kCommitChunk;
    const ChunkEntries ce = chunk_entries(b, h.n_ent, p0, lds);
    uint64_t key[kCommitU];
    uint32_t grp[kCommitU], inst[kCommitU], res[kCommitU];
#pragma unroll
    for (int u = 0; u < kCommitU; ++u) {
      const uint32_t p = p0 + u * kCommitThreads + threadIdx.x;
      key[u] = 0ull;
      grp[u] = inst[u] = 0u;
      res[u] = kPosZero;
      if (p >= h.n_pos) continue;
      const uint32_t e = entry_of(b, h.n_ent, ce, lds, p);
      const int32_t j = (int32_t)(p - b.ent_off[e]);
      const ps_req q = b.reqs[b.ent_req[e]];
      const ChainRef c{b.pool + q.pre_off, b.pool + q.tail_off, q.pre_len, q.pre_len + q.tail_len};
      grp[u] = b.ent_grp[e];
      inst[u] = (uint32_t)b.grp_inst[grp[u]];
      if (b.ent_skip && (uint32_t)j < b.ent_skip[e]) res[u] = kPosOld;
      else key[u] = chain_global(c, j);
    }
    Bucket bk[kCommitU];
    uint32_t bkt[kCommitU];
#pragma unroll
    for (int u = 0; u < kCommitU; ++u) {
      bkt[u] = bucket_of(key[u], inst[u], b.t.shift);
      bk[u] = Bucket{};
      if (key[u] != 0ull)
        bk[u] = load_bucket(table_of(b.t, inst[u]) + (size_t)bkt[u] * kSlotsPerBucket);
    }
#pragma unroll
    for (int u = 0; u < kCommitU; ++u) {
      const uint32_t p = p0 + u * kCommitThreads + threadIdx.x;
      if (p >= h.n_pos) continue;
      if (key[u] != 0ull) {
        uint32_t st = lane_status(bk[u], key[u]);
        if (st == 2u) st = lane_resolve(b.t, table_of(b.t, inst[u]), bkt[u], key[u]) ? 1u : 0u;
        if (st == 1u) {
          res[u] = kPosOld;
        } else {
          const uint32_t g0 = b.ent_off[b.grp_ent[grp[u]]], g1 = b.ent_off[b.grp_ent[grp[u] + 1]];
          const uint32_t slot = set_claim(b.set_key, 2u * g0, 2u * (g1 - g0), key[u]);
          // (positions only fall: a stale read at or below p is enough)
          if (b.set_pos[slot] > p) atomicMin(&b.set_pos[slot], p);
          res[u] = slot;
        }
      }
      b.pos_slot[p] = res[u];
    }
  }
}

// Hits (least position without its block) and the first occurrences per
// chunk.
__global__ __launch_bounds__(kCommitThreads) void commit_mark_kernel(CommitBatch b) {
  __shared__ uint32_t lds[kOffLds];
  __shared__ uint32_t total;
  const CommitHdr h = *b.hdr;
  const int lane = threadIdx.x & 63;
  const uint32_t chunks = (h.n_pos + kCommitChunk - 1) / kCommitChunk;
  for (uint32_t ch = blockIdx.x; ch < chunks; ch += gridDim.x) {
    const uint32_t p0 = ch * kCommitChunk;
    if (threadIdx.x == 0) total = 0u;
    const ChunkEntries ce = chunk_entries(b, h.n_ent, p0, lds);
    uint32_t n_won = 0;
    uint32_t slot[kCommitU], pos[kCommitU];
#pragma unroll
    for (int u = 0; u < kCommitU; ++u) {
      const uint32_t p = p0 + u * kCommitThreads + threadIdx.x;
      slot[u] = p < h.n_pos ? b.pos_slot[p] : kPosOld;
    }
#pragma unroll
    for (int u = 0; u < kCommitU; ++u) pos[u] = slot[u] < kPosZero ? b.set_pos[slot[u]] : 0u;
#pragma unroll
    for (int u = 0; u < kCommitU; ++u) {
      const uint32_t p = p0 + u * kCommitThreads + threadIdx.x;
      const bool in = p < h.n_pos;
      uint32_t e = 0u, j = 0u;
      bool miss = false;
      if (in) {
        e = entry_of(b, h.n_ent, ce, lds, p);
        const uint32_t e_off = b.ent_off[e];
        j = p - e_off;
        miss = slot[u] == kPosZero || (slot[u] < kPosZero && pos[u] >= e_off);
      }
      const bool won = in && slot[u] < kPosZero && pos[u] == p;
      n_won += (uint32_t)__popcll(__ballot(won));
      // one atomic per wave and entry run: the lowest missing lane of the
      // wave, and any lane that starts another entry's misses
      const uint64_t mm = __ballot(miss);
      const uint32_t e_prev = (uint32_t)__shfl_up((int)e, 1);
      const bool first = miss && (lane == 0 || !((mm >> (lane - 1)) & 1ull) || e_prev != e);
      if (first && j < b.ent_hit[e]) atomicMin(&b.ent_hit[e], j);
    }
    if (lane == 0 && n_won) atomicAdd(&total, n_won);
    __syncthreads();
    if (threadIdx.x == 0) b.chunk_won[ch] = total;
  }
}

// Exclusive scan of the chunk counts (one workgroup).
__global__ __launch_bounds__(1024) void commit_scan_kernel(CommitBatch b) {
  __shared__ uint32_t part[16];
  const CommitHdr h = *b.hdr;
  const uint32_t chunks = (h.n_pos + kCommitChunk - 1) / kCommitChunk;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  uint32_t run = 0;
  for (uint32_t c0 = 0; c0 < chunks; c0 += 1024) {
    const uint32_t c = c0 + threadIdx.x;
    const uint32_t v = c < chunks ? b.chunk_won[c] : 0u;
    const uint32_t ex = wave_exclusive_sum(v, lane);
    if (lane == 63) part[wv] = ex + v;
    __syncthreads();
    uint32_t before = run, all = 0;
    for (int k = 0; k < 16; ++k) {
      if (k < wv) before += part[k];
      all += part[k];
    }
    if (c < chunks) b.chunk_won[c] = before + ex;
    run += all;
    __syncthreads();
  }
  if (threadIdx.x == 0) b.chunk_won[chunks] = run;
}

// First occurrences before position p (every lane of the wave calls it).
__device__ uint32_t rank_at(const CommitBatch& b, uint32_t n_pos, uint32_t p, int lane) {
  const uint32_t ch = p / kCommitChunk;
  uint32_t r = b.chunk_won[ch];
  for (uint32_t k = ch * kCommitChunk; k < p; k += 64 * kCommitU) {
    uint32_t s[kCommitU], w[kCommitU];
#pragma unroll
    for (int u = 0; u < kCommitU; ++u) {
      const uint32_t x = k + 64u * u + (uint32_t)lane;
      s[u] = x < p && x < n_pos ? b.pos_slot[x] : kPosOld;
    }
#pragma unroll
    for (int u = 0; u < kCommitU; ++u) w[u] = s[u] < kPosZero ? b.set_pos[s[u]] : 0u;
#pragma unroll
    for (int u = 0; u < kCommitU; ++u)
      r += (uint32_t)__popcll(__ballot(s[u] < kPosZero && w[u] == k + 64u * u + (uint32_t)lane));
  }
  return r;
}

// One wave per group (instance): first occurrences before its bounds, and the
// row length they leave.
__global__ __launch_bounds__(64) void commit_group_kernel(CommitBatch b) {
  const CommitHdr h = *b.hdr;
  const int lane = threadIdx.x;
  for (uint32_t g = blockIdx.x; g < h.n_grp; g += gridDim.x) {
    const uint32_t e0 = b.grp_ent[g], e1 = b.grp_ent[g + 1];
    const uint32_t inst = (uint32_t)b.grp_inst[g];
    const uint32_t r0 = rank_at(b, h.n_pos, b.ent_off[e0], lane);
    const uint32_t r1 = rank_at(b, h.n_pos, b.ent_off[e1], lane);
    const uint32_t count0 = b.t.count[inst];
    const uint32_t room = b.cap > count0 ? b.cap - count0 : 0u;
    const uint32_t n_new = r1 - r0 < room ? r1 - r0 : room;
    if (lane == 0) {
      b.grp_rank[g] = r0;
      b.grp_count[g] = count0;
      b.t.count[inst] = count0 + n_new;
      if (r1 - r0 > room) *b.cap_binds = 1u;
    }
  }
}

// First occurrences inside the room enter the table and the row.
__global__ __launch_bounds__(kCommitThreads) void commit_insert_kernel(CommitBatch b) {
  __shared__ uint32_t lds[kOffLds];
  __shared__ uint32_t cnt[kCommitU][kCommitThreads / 64];
  const CommitHdr h = *b.hdr;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const uint64_t lt_mask = (1ull << lane) - 1ull;
  const uint32_t chunks = (h.n_pos + kCommitChunk - 1) / kCommitChunk;
  for (uint32_t ch = blockIdx.x; ch < chunks; ch += gridDim.x) {
    const uint32_t p0 = ch * kCommitChunk;
    const uint32_t rank0 = b.chunk_won[ch];
    if (b.chunk_won[ch + 1] == rank0) continue;  // nothing new in the chunk (workgroup-uniform)
    const ChunkEntries ce = chunk_entries(b, h.n_ent, p0, lds);
    uint32_t slot[kCommitU], rk[kCommitU];
    bool won[kCommitU];
#pragma unroll
    for (int u = 0; u < kCommitU; ++u) {
      const uint32_t p = p0 + u * kCommitThreads + threadIdx.x;
      slot[u] = p < h.n_pos ? b.pos_slot[p] : kPosOld;
    }
#pragma unroll
    for (int u = 0; u < kCommitU; ++u) {
      const uint32_t p = p0 + u * kCommitThreads + threadIdx.x;
      won[u] = slot[u] < kPosZero && b.set_pos[slot[u]] == p;
    }
#pragma unroll
    for (int u = 0; u < kCommitU; ++u) {
      const uint64_t wm = __ballot(won[u]);
      rk[u] = (uint32_t)__popcll(wm & lt_mask);
      if (lane == 0) cnt[u][wv] = (uint32_t)__popcll(wm);
    }
    __syncthreads();
    uint32_t run = rank0;
#pragma unroll
    for (int u = 0; u < kCommitU; ++u) {
      for (int k = 0; k < kCommitThreads / 64; ++k) {
        if (k == wv) rk[u] += run;
        run += cnt[u][k];
      }
    }
    uint64_t key[kCommitU];
    uint32_t inst[kCommitU], at[kCommitU];
    bool ins[kCommitU];
#pragma unroll
    for (int u = 0; u < kCommitU; ++u) {
      const uint32_t p = p0 + u * kCommitThreads + threadIdx.x;
      key[u] = 0ull;
      inst[u] = at[u] = 0u;
      ins[u] = false;
      if (!won[u]) continue;
      const uint32_t e = entry_of(b, h.n_ent, ce, lds, p);
      const uint32_t g = b.ent_grp[e];
      const uint32_t r = rk[u] - b.grp_rank[g];
      key[u] = b.set_key[slot[u]];
      b.set_key[slot[u]] = r;  // for the drop kernel (here only the winner reads its slot)
      inst[u] = (uint32_t)b.grp_inst[g];
      at[u] = b.grp_count[g] + r;
      ins[u] = at[u] < b.cap;
    }
#pragma unroll
    for (int u = 0; u < kCommitU; ++u) {
      if (!ins[u]) continue;
      uint32_t s = 0;
      (void)insert_key(b.t, inst[u], key[u], &s);
      b.t.rows[(size_t)inst[u] * (size_t)b.t.row_cap + at[u]] = key[u];
      b.t.rowpos[(size_t)inst[u] * (size_t)b.t.slots + s] = at[u];
    }
  }
}

// Refused positions: every position whose block's first occurrence ranked
// past the room; the block never becomes present, so it ends its entry's hit
// too.  Runs only where some group's cap binds.
__global__ __launch_bounds__(kCommitThreads) void commit_drop_kernel(CommitBatch b) {
  __shared__ uint32_t lds[kOffLds];
  if (*b.cap_binds == 0u) return;
  const CommitHdr h = *b.hdr;
  const int lane = threadIdx.x & 63;
  const uint32_t chunks = (h.n_pos + kCommitChunk - 1) / kCommitChunk;
  unsigned long long n = 0;
  for (uint32_t ch = blockIdx.x; ch < chunks; ch += gridDim.x) {
    const uint32_t p0 = ch * kCommitChunk;
    const ChunkEntries ce = chunk_entries(b, h.n_ent, p0, lds);
#pragma unroll
    for (int u = 0; u < kCommitU; ++u) {
      const uint32_t p = p0 + u * kCommitThreads + threadIdx.x;
      bool refused = false;
      uint32_t ent = 0u, at = 0u;
      if (p < h.n_pos) {
        const uint32_t s = b.pos_slot[p];
        if (s < kPosZero) {
          const uint32_t e = entry_of(b, h.n_ent, ce, lds, p);
          refused = b.grp_count[b.ent_grp[e]] + (uint32_t)b.set_key[s] >= b.cap;
          const uint32_t j = p - b.ent_off[e];
          ent = e;
          at = j;
        }
      }
      const uint64_t rm = __ballot(refused);
      n += (unsigned long long)__popcll(rm);
      // (one atomic per wave and entry: positions ascend with the lanes)
      const uint32_t e_prev = (uint32_t)__shfl_up((int)ent, 1);
      const bool first = refused && (lane == 0 || !((rm >> (lane - 1)) & 1ull) || e_prev != ent);
      if (first && at < b.ent_hit[ent]) atomicMin(&b.ent_hit[ent], at);
    }
  }
  if (lane == 0 && n) atomicAdd(b.dropped, n);
}

// One wave per group: the instance's counters as its entries move them.
__global__ __launch_bounds__(64) void commit_state_kernel(CommitBatch b) {
  const CommitHdr h = *b.hdr;
  const int lane = threadIdx.x;
  const DevModel& m = *b.model;
  for (uint32_t g = blockIdx.x; g < h.n_grp; g += gridDim.x) {
    const uint32_t e0 = b.grp_ent[g], e1 = b.grp_ent[g + 1];
    const uint32_t inst = (uint32_t)b.grp_inst[g];
    // uncached and total tokens of the entries (blocks: 64-bit sums)
    unsigned long long uncached = 0, blocks = 0;
    for (uint32_t e = e0 + (uint32_t)lane; e < e1; e += 64) {
      const uint32_t len = b.ent_off[e + 1] - b.ent_off[e];
      blocks += len;
      uncached += len - b.ent_hit[e];
    }
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) {
      blocks += __shfl_xor(blocks, d);
      uncached += __shfl_xor(uncached, d);
    }
    if (lane == 0) {
      InstState st = b.inst[inst];
      const int32_t n = (int32_t)(e1 - e0);
      st.Q += n;
      st.A1 += n;
      st.P += (int64_t)uncached * m.bs;
      st.S += (int64_t)blocks * m.bs;
      st.seg = segment_of(m, st.A1);
      b.inst[inst] = st;
      b.room[inst] = st.A1 <= m.b_max ? m.kv_cap - st.S : -1;
    }
  }
}

}  // namespace

// The workspace of a batch of at most n_ent entries and n_pos positions.
size_t ps_commit_ws_bytes(uint32_t n_ent, uint32_t n_grp, uint32_t n_pos) {
  return (size_t)n_pos * kCommitPosBytes +
         ((size_t)n_pos / kCommitChunk + 2) * sizeof(uint32_t) + (size_t)n_ent * sizeof(uint32_t) +
         2 * (size_t)n_grp * sizeof(uint32_t) + 16 * 256;
}

void ps_commit_ws_bind(CommitBatch* b, void* ws, uint32_t n_ent, uint32_t n_grp, uint32_t n_pos) {
  unsigned char* p = (unsigned char*)ws;
  auto take = [&](size_t bytes) {
    void* r = p;
    p += (bytes + 255) & ~(size_t)255;
    return r;
  };
  b->set_key = (unsigned long long*)take(2 * (size_t)n_pos * sizeof(uint64_t));
  b->set_pos = (uint32_t*)take(2 * (size_t)n_pos * sizeof(uint32_t));
  b->pos_slot = (uint32_t*)take((size_t)n_pos * sizeof(uint32_t));
  b->chunk_won = (uint32_t*)take(((size_t)n_pos / kCommitChunk + 2) * sizeof(uint32_t));
  b->ent_hit = (uint32_t*)take((size_t)n_ent * sizeof(uint32_t));
  b->grp_rank = (uint32_t*)take((size_t)n_grp * sizeof(uint32_t));
  b->grp_count = (uint32_t*)take((size_t)n_grp * sizeof(uint32_t));
  b->cap_binds = (uint32_t*)take(sizeof(uint32_t));
}

hipError_t ps_launch_commit(const CommitBatch& b, uint32_t max_grp, uint32_t max_pos, hipStream_t s) {
  // grids for the largest batch the caller may have put behind hdr; the
  // kernels stride over what is there
  const unsigned chunks = (unsigned)((max_pos + kCommitChunk - 1) / kCommitChunk);
  const unsigned grid = chunks < 1u ? 1u : (chunks < 8192u ? chunks : 8192u);
  const unsigned ggrid = max_grp < 1u ? 1u : (max_grp < 4096u ? max_grp : 4096u);
  hipLaunchKernelGGL(commit_clear_kernel, dim3(grid), dim3(kCommitThreads), 0, s, b);
  hipLaunchKernelGGL(commit_probe_kernel, dim3(grid), dim3(kCommitThreads), 0, s, b);
  hipLaunchKernelGGL(commit_mark_kernel, dim3(grid), dim3(kCommitThreads), 0, s, b);
  hipLaunchKernelGGL(commit_scan_kernel, dim3(1), dim3(1024), 0, s, b);
  hipLaunchKernelGGL(commit_group_kernel, dim3(ggrid), dim3(64), 0, s, b);
  hipLaunchKernelGGL(commit_insert_kernel, dim3(grid), dim3(kCommitThreads), 0, s, b);
  hipLaunchKernelGGL(commit_drop_kernel, dim3(grid), dim3(kCommitThreads), 0, s, b);
  if (b.move_state) hipLaunchKernelGGL(commit_state_kernel, dim3(ggrid), dim3(64), 0, s, b);
  return hipGetLastError();
}
