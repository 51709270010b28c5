// Prefix index build: all (block hash, instance) pairs of the instances'
// rows, sorted by the index hash with hipCUB's radix sort (stable, so each
// block's holders stay in ascending instance order); the runs of equal keys
// then come in bucket order and go to the open-addressing table of 16-byte
// entries by a running maximum.  Runs at ps_load_instances and after commits.

#include <hipcub/hipcub.hpp>

#include <vector>

#include "ps_common.h"

using namespace ps;

namespace {

// The index hash before its shift to a bucket (bucket_of with kIndexSalt): a
// bijection of the 64-bit keys, so sorting by it groups equal keys and puts
// the distinct ones in bucket order at once.
constexpr uint64_t kIdxXor = 0x9E3779B97F4A7C15ull * (uint64_t)(kIndexSalt + 1u);
constexpr uint64_t kIdxMul = 0xD6E8FEB86659FD93ull;
constexpr uint64_t inverse64(uint64_t a) {  // a odd: Newton's iteration mod 2^64
  uint64_t x = a;
  for (int k = 0; k < 6; ++k) x *= 2ull - a * x;
  return x;
}
constexpr uint64_t kIdxInv = inverse64(kIdxMul);
static_assert(kIdxInv * kIdxMul == 1ull, "inverse of the index multiplier");

constexpr int kIdxThreads = 256;
constexpr int kIdxU = 8;
constexpr uint32_t kIdxChunk = kIdxThreads * kIdxU;

// Pairs of instance i at [base[i], base[i + 1]), from its row: a straight
// copy.  (Scanning the hash tables for occupied slots read at least twice the
// slots for the keys and took an atomic per wave: 1.2 ms at 64 tables of
// 131,072 slots, 2.1 ms at 1,024; this takes 10 us.)
__global__ __launch_bounds__(kIdxThreads) void extract_kernel(Tables t, const int64_t* base, uint64_t* pk,
                                                              uint16_t* pv) {
  const uint32_t i = blockIdx.x;
  const int64_t b = base[i], n = base[i + 1] - b;
  const uint64_t* row = t.rows + (size_t)i * (size_t)t.row_cap;
  for (int64_t k = (int64_t)blockIdx.y * kIdxChunk + threadIdx.x; k < n; k += (int64_t)gridDim.y * kIdxChunk) {
    uint64_t v[kIdxU];
#pragma unroll
    for (int u = 0; u < kIdxU; ++u) v[u] = k + u * kIdxThreads < n ? row[k + u * kIdxThreads] : 0ull;
#pragma unroll
    for (int u = 0; u < kIdxU; ++u) {
      if (k + u * kIdxThreads >= n) continue;
      pk[b + k + u * kIdxThreads] = (v[u] ^ kIdxXor) * kIdxMul;
      pv[b + k + u * kIdxThreads] = (uint16_t)i;
    }
  }
}

// Runs of equal keys and, among them, the popular ones (more than kPopular
// long), per chunk of sorted pairs.
__global__ __launch_bounds__(kIdxThreads) void run_count_kernel(const uint64_t* sk, uint32_t n, uint2* cnt) {
  __shared__ uint32_t heads, pops;
  if (threadIdx.x == 0) heads = pops = 0u;
  __syncthreads();
  uint32_t nh = 0, np = 0;
#pragma unroll
  for (int u = 0; u < kIdxU; ++u) {
    const uint32_t i = blockIdx.x * kIdxChunk + u * kIdxThreads + threadIdx.x;
    const bool head = i < n && (i == 0 || sk[i] != sk[i - 1]);
    const bool pop = head && n - i > kPopular && sk[i + kPopular] == sk[i];
    nh += (uint32_t)__popcll(__ballot(head));
    np += (uint32_t)__popcll(__ballot(pop));
  }
  if ((threadIdx.x & 63) == 0) {
    atomicAdd(&heads, nh);
    atomicAdd(&pops, np);
  }
  __syncthreads();
  if (threadIdx.x == 0) cnt[blockIdx.x] = make_uint2(heads, pops);
}

// Exclusive sums of the chunk counts, in place; the totals in cnt[chunks]
// (one workgroup).
__global__ __launch_bounds__(1024) void run_scan_kernel(uint2* cnt, uint32_t chunks) {
  __shared__ uint2 part[16];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  uint2 run = make_uint2(0u, 0u);
  for (uint32_t c0 = 0; c0 < chunks; c0 += 1024) {
    const uint32_t c = c0 + threadIdx.x;
    const uint2 v = c < chunks ? cnt[c] : make_uint2(0u, 0u);
    const uint32_t ex = wave_exclusive_sum(v.x, lane), ey = wave_exclusive_sum(v.y, lane);
    if (lane == 63) part[wv] = make_uint2(ex + v.x, ey + v.y);
    __syncthreads();
    uint2 before = run;
    for (int k = 0; k < 16; ++k) {
      if (k < wv) {
        before.x += part[k].x;
        before.y += part[k].y;
      }
      run.x += part[k].x;
      run.y += part[k].y;
    }
    if (c < chunks) cnt[c] = make_uint2(before.x + ex, before.y + ey);
    __syncthreads();
  }
  if (threadIdx.x == 0) cnt[chunks] = run;
}

// Start of every run (rs[run], rs[n_runs] = n), its popular rank (~0: a list)
// and the popular runs' numbers.
__global__ __launch_bounds__(kIdxThreads) void run_place_kernel(const uint64_t* sk, uint32_t n, const uint2* cnt,
                                                                uint32_t chunks, uint32_t* rs, uint32_t* prank,
                                                                uint32_t* prun) {
  __shared__ uint2 part[kIdxU][kIdxThreads / 64];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const uint64_t lt = (1ull << lane) - 1ull;
  uint64_t hm[kIdxU], pm[kIdxU];
#pragma unroll
  for (int u = 0; u < kIdxU; ++u) {
    const uint32_t i = blockIdx.x * kIdxChunk + u * kIdxThreads + threadIdx.x;
    const bool head = i < n && (i == 0 || sk[i] != sk[i - 1]);
    const bool pop = head && n - i > kPopular && sk[i + kPopular] == sk[i];
    hm[u] = __ballot(head);
    pm[u] = __ballot(pop);
    if (lane == 0) part[u][wv] = make_uint2((uint32_t)__popcll(hm[u]), (uint32_t)__popcll(pm[u]));
  }
  __syncthreads();
  uint2 run = cnt[blockIdx.x];
#pragma unroll
  for (int u = 0; u < kIdxU; ++u) {
    const uint32_t i = blockIdx.x * kIdxChunk + u * kIdxThreads + threadIdx.x;
    for (int k = 0; k < kIdxThreads / 64; ++k) {
      if (k == wv && ((hm[u] >> lane) & 1ull)) {
        const uint32_t r = run.x + (uint32_t)__popcll(hm[u] & lt);
        rs[r] = i;
        const bool pop = ((pm[u] >> lane) & 1ull) != 0ull;
        const uint32_t pr = run.y + (uint32_t)__popcll(pm[u] & lt);
        prank[r] = pop ? pr : ~0u;
        if (pop) prun[pr] = r;
      }
      run.x += part[u][k].x;
      run.y += part[u][k].y;
    }
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) rs[cnt[chunks].x] = n;
}

// Linear probing over buckets, without a probe: the runs come in bucket
// order, so run k goes to slot max(8 * its bucket, slot of run k - 1, plus
// one) = k + max over j <= k of (8 * bucket_j - j).  Maximum per chunk of
// runs, then a running maximum of those (one workgroup), then every run's
// slot.  (Compare-and-swap inserts of unsorted keys wrote one 128-byte line
// at a time through the memory side: 0.92 ms at 6 M keys, 5.7 ms at 45 M.)
__device__ __forceinline__ int64_t slot_lead(const uint64_t* sk, const uint32_t* rs, uint32_t k, uint32_t shift) {
  const uint64_t b = shift >= 64 ? 0ull : sk[rs[k]] >> shift;
  return (int64_t)(b * kSlotsPerBucket) - (int64_t)k;
}

__device__ __forceinline__ int64_t wave_inclusive_max(int64_t v, int lane) {
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int64_t y = __shfl_up(v, d);
    if (lane >= d && y > v) v = y;
  }
  return v;
}

__global__ __launch_bounds__(kIdxThreads) void lead_kernel(const uint64_t* sk, const uint32_t* rs, uint32_t runs,
                                                           uint32_t shift, int64_t* lead) {
  __shared__ int64_t part[kIdxThreads / 64];
  int64_t v = INT64_MIN;
#pragma unroll
  for (int u = 0; u < kIdxU; ++u) {
    const uint32_t k = blockIdx.x * kIdxChunk + u * kIdxThreads + threadIdx.x;
    if (k < runs) {
      const int64_t x = slot_lead(sk, rs, k, shift);
      v = x > v ? x : v;
    }
  }
  v = wave_inclusive_max(v, threadIdx.x & 63);
  if ((threadIdx.x & 63) == 63) part[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int k = 1; k < kIdxThreads / 64; ++k) v = part[k] > part[k - 1] ? part[k] : (part[k] = part[k - 1]);
    lead[blockIdx.x] = part[kIdxThreads / 64 - 1];
  }
}

__global__ __launch_bounds__(1024) void lead_scan_kernel(int64_t* lead, uint32_t chunks) {
  __shared__ int64_t part[16];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  int64_t run = INT64_MIN;
  for (uint32_t c0 = 0; c0 < chunks; c0 += 1024) {
    const uint32_t c = c0 + threadIdx.x;
    const int64_t v = wave_inclusive_max(c < chunks ? lead[c] : INT64_MIN, lane);
    if (lane == 63) part[wv] = v;
    const int64_t left = __shfl_up(v, 1);
    __syncthreads();
    int64_t before = run;
    for (int k = 0; k < 16; ++k) {
      if (k < wv && part[k] > before) before = part[k];
      if (part[k] > run) run = part[k];
    }
    if (lane > 0 && left > before) before = left;
    if (c < chunks) lead[c] = before;  // maximum over the chunks before c
    __syncthreads();
  }
}

__device__ __forceinline__ IdxEntry run_entry(const uint64_t* sk, const uint32_t* rs, const uint32_t* prank,
                                              uint32_t k) {
  const uint32_t at = rs[k];
  const uint32_t pr = prank[k];
  return IdxEntry{(sk[at] * kIdxInv) ^ kIdxXor, pr != ~0u ? pr : at, rs[k + 1] - at};
}

__global__ __launch_bounds__(kIdxThreads) void index_place_kernel(GIndex x, const uint64_t* sk, const uint32_t* rs,
                                                                  const uint32_t* prank, uint32_t runs,
                                                                  const int64_t* lead) {
  __shared__ int64_t part[kIdxU][kIdxThreads / 64];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int64_t slots = ((int64_t)x.bmask + 1) * kSlotsPerBucket;
  int64_t v[kIdxU];
#pragma unroll
  for (int u = 0; u < kIdxU; ++u) {
    const uint32_t k = blockIdx.x * kIdxChunk + u * kIdxThreads + threadIdx.x;
    v[u] = wave_inclusive_max(k < runs ? slot_lead(sk, rs, k, x.shift) : INT64_MIN, lane);
    if (lane == 63) part[u][wv] = v[u];
  }
  __syncthreads();
  int64_t run = lead[blockIdx.x];
#pragma unroll
  for (int u = 0; u < kIdxU; ++u) {
    int64_t before = run;
    for (int k = 0; k < kIdxThreads / 64; ++k) {
      if (k < wv && part[u][k] > before) before = part[u][k];
      if (part[u][k] > run) run = part[u][k];
    }
    const uint32_t k = blockIdx.x * kIdxChunk + u * kIdxThreads + threadIdx.x;
    if (k >= runs) continue;
    const int64_t slot = (int64_t)k + (v[u] > before ? v[u] : before);
    if (slot < slots) x.ent[slot] = run_entry(sk, rs, prank, k);
  }
}

// The runs whose slot lies past the table's end go on at its first bucket
// (the slots from their own bucket to the end are full).  Slots ascend, so
// they are a suffix of the runs; one wave takes them in order.
__global__ __launch_bounds__(64) void index_wrap_kernel(GIndex x, const uint64_t* sk, const uint32_t* rs,
                                                        const uint32_t* prank, uint32_t runs, const int64_t* lead,
                                                        uint32_t chunks) {
  const int64_t slots = ((int64_t)x.bmask + 1) * kSlotsPerBucket;
  const int lane = threadIdx.x;
  // the last chunk that begins inside the table
  uint32_t c = chunks - 1;
  while (c > 0) {
    const uint32_t f = c * kIdxChunk;
    const int64_t lf = slot_lead(sk, rs, f, x.shift);
    if ((int64_t)f + (lead[c] > lf ? lead[c] : lf) < slots) break;
    --c;
  }
  int64_t run = lead[c];
  if (c == chunks - 1) {  // no run past the end (the usual case): one pass of loads in flight together
    int64_t m = run;
    uint32_t at[kIdxChunk / 64];
#pragma unroll
    for (int u = 0; u < (int)kIdxChunk / 64; ++u) {
      const uint32_t k = c * kIdxChunk + u * 64 + lane;
      at[u] = k < runs ? rs[k] : 0u;
    }
#pragma unroll
    for (int u = 0; u < (int)kIdxChunk / 64; ++u) {
      const uint32_t k = c * kIdxChunk + u * 64 + lane;
      const uint64_t b = x.shift >= 64 ? 0ull : sk[at[u]] >> x.shift;
      const int64_t v = (int64_t)(b * kSlotsPerBucket) - (int64_t)k;
      if (k < runs && v > m) m = v;
    }
    m = __shfl(wave_inclusive_max(m, lane), 63);
    if ((int64_t)runs - 1 + m < slots) return;
  }
  uint32_t free_slot = 0;
  for (uint32_t b = c * kIdxChunk; b < runs; b += 64) {
    const uint32_t k = b + (uint32_t)lane;
    int64_t v = wave_inclusive_max(k < runs ? slot_lead(sk, rs, k, x.shift) : INT64_MIN, lane);
    if (run > v) v = run;
    run = __shfl(v, 63);
    uint64_t past = __ballot(k < runs && (int64_t)k + v >= slots);
    while (past) {  // rare: one lane after the other
      const int l = __builtin_ctzll(past);
      past &= past - 1;
      while ((int64_t)free_slot < slots && x.ent[free_slot].key != 0ull) ++free_slot;
      if (lane == l && (int64_t)free_slot < slots) x.ent[free_slot] = run_entry(sk, rs, prank, k);
      ++free_slot;
    }
  }
}

// Holder bitmaps of the popular runs, a wave each: the bits gathered in LDS,
// then every word written once (no clearing before).  (A thread per run with
// an atomic per holder took 0.7 ms for 128 blocks of 1,000 holders.)
__global__ __launch_bounds__(64) void bitmap_kernel(GIndex x, const uint32_t* rs, const uint32_t* prun,
                                                    uint32_t n_pop) {
  extern __shared__ __align__(16) unsigned char smem[];
  uint32_t* w = reinterpret_cast<uint32_t*>(smem);
  for (uint32_t p = blockIdx.x; p < n_pop; p += gridDim.x) {
    const uint32_t r = prun[p], a = rs[r], b = rs[r + 1];
    for (uint32_t k = threadIdx.x; k < 2 * x.nw; k += 64) w[k] = 0u;
    __syncthreads();
    for (uint32_t k = a + threadIdx.x; k < b; k += 64) {
      const uint32_t id = x.holders[k];
      atomicOr(&w[id >> 5], 1u << (id & 31u));
    }
    __syncthreads();
    uint32_t* bm = reinterpret_cast<uint32_t*>(x.bitmaps + (size_t)p * x.nw);
    for (uint32_t k = threadIdx.x; k < 2 * x.nw; k += 64) bm[k] = w[k];
    __syncthreads();
  }
}

}  // namespace

void ps_free_index(GIndex* x, DevPool* pool) {
  pool->put(x->ent, x->holders, x->bitmaps);
  x->bmask = 0;
  x->shift = 64;
}

#define TRY(call)                   \
  do {                              \
    e = (call);                     \
    if (e != hipSuccess) goto done; \
  } while (0)

hipError_t ps_build_index(const Tables& t, int32_t n_inst, const uint32_t* count_host, GIndex* x,
                          DevPool* pool, hipStream_t s) {
  hipError_t e = hipSuccess;
  std::vector<int64_t> base((size_t)n_inst + 1, 0);
  uint32_t longest = 0;
  for (int32_t i = 0; i < n_inst; ++i) {
    base[(size_t)i + 1] = base[(size_t)i] + count_host[i];
    longest = std::max(longest, count_host[i]);
  }
  const int64_t n = base[(size_t)n_inst];
  if (n > (int64_t)INT32_MAX) return hipErrorInvalidValue;
  const uint32_t chunks = (uint32_t)((n + kIdxChunk - 1) / kIdxChunk);
  int64_t* d_base = nullptr;
  uint64_t *pk = nullptr, *sk = nullptr;
  uint16_t *pv = nullptr, *sv = nullptr;
  uint32_t *rs = nullptr, *prank = nullptr, *prun = nullptr;
  uint2* cnt = nullptr;
  int64_t* lead = nullptr;
  void* tmp = nullptr;
  size_t tmp_bytes = 0;
  uint2 tot = make_uint2(0u, 0u);  // distinct keys, popular ones
  GIndex nx{nullptr, nullptr, nullptr, (uint32_t)((n_inst + 63) / 64), 0, 64, 0};
  const size_t nn = (size_t)(n > 0 ? n : 1);
  int64_t buckets = 1;
  int log2b = 0;

  TRY(pool->get(&sv, nn * sizeof(uint16_t)));
  if (n > 0) {
    TRY(pool->get(&d_base, base.size() * sizeof(int64_t)));
    TRY(pool->get(&pk, nn * sizeof(uint64_t)));
    TRY(pool->get(&sk, nn * sizeof(uint64_t)));
    TRY(pool->get(&pv, nn * sizeof(uint16_t)));
    TRY(pool->get(&cnt, ((size_t)chunks + 1) * sizeof(uint2)));
    TRY(hipMemcpyAsync(d_base, base.data(), base.size() * sizeof(int64_t), hipMemcpyHostToDevice, s));
    const uint32_t row_chunks = std::min((longest + kIdxChunk - 1) / kIdxChunk, 1024u);
    hipLaunchKernelGGL(extract_kernel, dim3((unsigned)n_inst, row_chunks), dim3(kIdxThreads), 0, s, t, d_base,
                       pk, pv);
    TRY(hipGetLastError());
    TRY(hipcub::DeviceRadixSort::SortPairs(nullptr, tmp_bytes, pk, sk, pv, sv, (int)n, 0, 64, s));
    TRY(pool->get(&tmp, tmp_bytes));
    TRY(hipcub::DeviceRadixSort::SortPairs(tmp, tmp_bytes, pk, sk, pv, sv, (int)n, 0, 64, s));
    hipLaunchKernelGGL(run_count_kernel, dim3(chunks), dim3(kIdxThreads), 0, s, sk, (uint32_t)n, cnt);
    hipLaunchKernelGGL(run_scan_kernel, dim3(1), dim3(1024), 0, s, cnt, chunks);
    TRY(hipGetLastError());
    TRY(hipMemcpyAsync(&tot, cnt + chunks, sizeof tot, hipMemcpyDeviceToHost, s));
    TRY(hipStreamSynchronize(s));
  }
  // table of >= 2 * runs entries in buckets of 8
  while (buckets * kSlotsPerBucket < 2 * (int64_t)tot.x) {
    buckets <<= 1;
    ++log2b;
  }
  nx.bmask = (uint32_t)(buckets - 1);
  nx.shift = (uint32_t)(64 - log2b);
  nx.n_pop = tot.y;
  TRY(pool->get(&nx.ent, (size_t)buckets * kSlotsPerBucket * sizeof(IdxEntry)));
  TRY(hipMemsetAsync(nx.ent, 0, (size_t)buckets * kSlotsPerBucket * sizeof(IdxEntry), s));
  if (tot.y > 0) TRY(pool->get(&nx.bitmaps, (size_t)tot.y * nx.nw * sizeof(uint64_t)));
  if (tot.x > 0) {
    const uint32_t rchunks = (tot.x + kIdxChunk - 1) / kIdxChunk;
    TRY(pool->get(&rs, ((size_t)tot.x + 1) * sizeof(uint32_t)));
    TRY(pool->get(&prank, (size_t)tot.x * sizeof(uint32_t)));
    TRY(pool->get(&prun, ((size_t)tot.y + 1) * sizeof(uint32_t)));
    TRY(pool->get(&lead, (size_t)rchunks * sizeof(int64_t)));
    hipLaunchKernelGGL(run_place_kernel, dim3(chunks), dim3(kIdxThreads), 0, s, sk, (uint32_t)n, cnt, chunks, rs,
                       prank, prun);
    hipLaunchKernelGGL(lead_kernel, dim3(rchunks), dim3(kIdxThreads), 0, s, sk, rs, tot.x, nx.shift, lead);
    hipLaunchKernelGGL(lead_scan_kernel, dim3(1), dim3(1024), 0, s, lead, rchunks);
    hipLaunchKernelGGL(index_place_kernel, dim3(rchunks), dim3(kIdxThreads), 0, s, nx, sk, rs, prank, tot.x, lead);
    hipLaunchKernelGGL(index_wrap_kernel, dim3(1), dim3(64), 0, s, nx, sk, rs, prank, tot.x, lead, rchunks);
    nx.holders = sv;  // read by bitmap_kernel
    if (tot.y > 0)
      hipLaunchKernelGGL(bitmap_kernel, dim3(std::min(tot.y, 4096u)), dim3(64), (size_t)nx.nw * sizeof(uint64_t), s,
                         nx, rs, prun, tot.y);
    TRY(hipGetLastError());
  }
  TRY(hipStreamSynchronize(s));
  nx.holders = sv;
  sv = nullptr;
  ps_free_index(x, pool);
  *x = nx;
  nx.ent = nullptr;
  nx.bitmaps = nullptr;
done:
  pool->put(nx.ent, nx.bitmaps, d_base, pk, sk, pv, sv, rs, prank, prun, cnt, lead, tmp);
  return e;
}

hipError_t ps_exclusive_scan_u32(const uint32_t* in, uint32_t* out, int64_t n, DevPool* pool,
                                 hipStream_t s) {
  if (n <= 0) return hipSuccess;
  size_t bytes = 0;
  hipError_t e = hipcub::DeviceScan::ExclusiveSum(nullptr, bytes, in, out, (int)n, s);
  if (e != hipSuccess) return e;
  void* tmp = nullptr;
  e = pool->get(&tmp, bytes);
  if (e != hipSuccess) return e;
  e = hipcub::DeviceScan::ExclusiveSum(tmp, bytes, in, out, (int)n, s);
  pool->put(tmp);
  return e;
}
