// Per-arrival scheduler in batches (Algorithm 1 taken one request at a time,
// each placement committed before the next request is scored).
//
// Requests are decided in order by one workgroup, so its time per decision is
// the scheduler's: what depends on the order has to be small and wait for
// nothing.  A kernel that also inserted every placed request's blocks before
// the next decision, and probed the changed instances' tables per request,
// took 16-20 us a decision (dependent reads: 14 us inserts, 5 us probes).
// Here a batch of up to kSpecBatch requests leaves the tables as they are:
//   plan    - the batch: next requests, their lengths;
//   first, walk - every request's hit on every instance, by table and row;
//   spec    - every request scored against the batch's starting state;
//   intern, check, lcp - how far two requests' chains agree;
//   decide  - in arrival order, from the above and the state of the instances
//             placed on so far, which is all that changed (LDS, registers);
//   commit  - the batch's blocks enter the tables together (ps_commit.hip).
// A request's hit on an instance that took an earlier request q of the batch
// is the least position whose block neither the table nor q's chain has.
// With chained hashes that is max(table hit, common prefix with q).  `check`
// makes sure: a block seen before in the batch must stand at the same
// position behind the same block (so equal blocks mean equal prefixes); the
// batch ends before the first request that breaks this, and where the table
// goes on behind the common prefix or the table's cap could refuse blocks,
// decide ends it too.  The next batch begins there.

#include <algorithm>

#include "ps_common.h"

namespace {

constexpr uint32_t kNone16 = 0xFFFFu;

// What a request does to the changed instances (or'ed over them).
constexpr uint32_t kMoved = 1u;    // the hit of one that is in A moved
constexpr uint32_t kBelow = 2u;    // one that is in A lies below the batch's W_min
constexpr uint32_t kMinThen = 4u;  // one was at W_min ...
constexpr uint32_t kMinNow = 8u;   // ... and one that is in A is

// ------------------------------------------------------------------- a batch
// The next batch: requests from the cursor on, at most max_n of them and (but
// for a single longer one) at most max_pos positions.
__global__ __launch_bounds__(kSpecBatch) void plan_kernel(SchedArgs a) {
  __shared__ uint32_t part[kSpecBatch / 64];
  const uint32_t r0 = *a.cursor;
  const uint32_t tid = threadIdx.x;
  const int lane = tid & 63, wv = tid >> 6;
  const uint32_t left = (uint32_t)a.n_req - r0;  // the cursor never passes n_req
  const uint32_t nb = left < a.max_n ? left : a.max_n;
  uint32_t len = 0u;
  bool ok = false;
  if (tid < nb) {
    const ps_req q = a.reqs[r0 + tid];
    ok = req_valid(q, a.pool_len);
    len = ok ? (uint32_t)(q.pre_len + q.tail_len) : 0u;
  }
  const uint32_t ex = wave_exclusive_sum(len, lane);
  if (lane == 63) part[wv] = ex + len;
  __syncthreads();
  uint64_t off = ex;  // at most kSpecBatch chains of 2^24 blocks: 2^32
  for (int k = 0; k < wv; ++k) off += part[k];
  const bool in = tid < nb && (tid == 0u || off + len <= a.max_pos);
  a.blen[tid] = ok ? len : ~0u;
  a.zero_at[tid] = len;
  a.off[tid] = (uint32_t)off;
  const uint64_t bm = __ballot(in);
  __syncthreads();
  if (lane == 0) part[wv] = (uint32_t)__popcll(bm);
  __syncthreads();
  uint32_t n = 0;
  for (int k = 0; k < kSpecBatch / 64; ++k) n += part[k];
  // (`in` holds for a prefix of the requests: offsets ascend)
  if (n == 0u ? tid == 0u : tid == n - 1u) {
    const uint32_t pos = n == 0u ? 0u : (uint32_t)off + len;
    a.off[n] = pos;
    *a.hdr = SchedHdr{r0, n, pos, n};
    *a.n_work = 0u;
  }
}

// First block of every request on every instance; the instances that hold it
// go to the walk list.
__global__ __launch_bounds__(256) void first_kernel(SchedArgs a) {
  const SchedHdr h = *a.hdr;
  const uint32_t b = blockIdx.x;
  if (b >= h.n) return;
  const uint32_t len = a.blen[b];
  if (len == ~0u) return;
  const int lane = threadIdx.x & 63;
  const ps_req q = a.reqs[h.r0 + b];
  const ChainRef c{a.pool + q.pre_off, a.pool + q.tail_off, q.pre_len, (int32_t)len};
  const uint64_t k0 = len > 0u ? chain_global(c, 0) : 0ull;
  for (int32_t i0 = (int32_t)blockIdx.y * 256; i0 < a.n_inst; i0 += (int32_t)gridDim.y * 256) {
    const int32_t i = i0 + (int32_t)threadIdx.x;
    bool held = false;
    if (i < a.n_inst) {
      if (k0 != 0ull) {
        const uint64_t* tab = table_of(a.t, (uint32_t)i);
        const uint32_t bkt = bucket_of(k0, (uint32_t)i, a.t.shift);
        const uint32_t st = lane_status(load_bucket(tab + (size_t)bkt * kSlotsPerBucket), k0);
        held = st == 1u || (st == 2u && lane_resolve(a.t, tab, bkt, k0));
      }
      a.hits[(size_t)b * sched_row_stride(a.n_inst) + (size_t)i] = held ? 1u : 0u;
    }
    const uint64_t bm = __ballot(held && len > 1u);
    if (bm) {
      uint32_t at = 0;
      if (lane == 0) at = atomicAdd(a.n_work, (uint32_t)__popcll(bm));
      at = (uint32_t)__shfl((int)at, 0);
      if (held && len > 1u) a.work[at + (uint32_t)__popcll(bm & ((1ull << lane) - 1ull))] = b << 16 | (uint32_t)i;
    }
  }
}

// A wave per instance found, along its row, 256 positions in a run's first step
// and 512 after it (17 us for 256 requests with about one holder
// each; walking all of a request's holders in one wave by table probes took 73
// us).
__global__ __launch_bounds__(64) void walk_kernel(SchedArgs a) {
  const uint32_t n = *a.n_work;
  const uint32_t r0 = a.hdr->r0;
  const int lane = threadIdx.x;
  for (uint32_t k = blockIdx.x; k < n; k += gridDim.x) {
    const uint32_t w = a.work[k];
    const uint32_t b = w >> 16, i = w & 0xFFFFu;
    const ps_req q = a.reqs[r0 + b];
    const ChainRef c{a.pool + q.pre_off, a.pool + q.tail_off, q.pre_len, q.pre_len + q.tail_len};
    const uint32_t hit = run_walk<false, 8>(a.t, i, c, nullptr, 0, lane >> 3, lane & 7);
    if (lane == 0) a.hits[(size_t)b * sched_row_stride(a.n_inst) + i] = hit;
  }
}

// ------------------------------------------------------- what chains share
// Request of the batch that owns position p.
__device__ __forceinline__ uint32_t batch_of(const uint32_t* off, uint32_t n, uint32_t p) {
  uint32_t lo = 0, hi = n;
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) >> 1;
    if (off[mid] <= p) lo = mid;
    else hi = mid;
  }
  return lo;
}

__global__ __launch_bounds__(256) void intern_clear_kernel(SchedArgs a) {
  const size_t slots = 2 * (size_t)a.hdr->n_pos;
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (size_t k = (size_t)blockIdx.x * blockDim.x + threadIdx.x; k < slots; k += stride) {
    a.set_key[k] = 0ull;
    a.set_pos[k] = 0xFFFFFFFFu;
  }
}

// Every block of the batch and the first position that carries it; a
// request's first zero hash.  Bound by two memory-side atomics per position
// (60 us for 256 chains of about 2,100 blocks).
constexpr uint32_t kPosNone = 0xFFFFFFFFu;

__global__ __launch_bounds__(256) void intern_kernel(SchedArgs a) {
  __shared__ uint32_t off[kSpecBatch + 1];
  const SchedHdr h = *a.hdr;
  for (uint32_t k = threadIdx.x; k < h.n; k += 256) off[k] = a.off[k];
  __syncthreads();
  const uint32_t size = 2u * h.n_pos;
  const uint32_t stride = gridDim.x * 256u;
  for (uint32_t p = blockIdx.x * 256u + threadIdx.x; p < h.n_pos; p += stride) {
    const uint32_t b = batch_of(off, h.n, p);
    const int32_t j = (int32_t)(p - off[b]);
    const ps_req q = a.reqs[h.r0 + b];
    const uint64_t key = chain_global(ChainRef{a.pool + q.pre_off, a.pool + q.tail_off, q.pre_len, 0}, j);
    uint32_t slot = kPosNone;
    if (key == 0ull) {
      atomicMin(&a.zero_at[b], (uint32_t)j);
    } else {
      uint32_t at = (uint32_t)((((key * 0x9E3779B97F4A7C15ull) >> 32) * (uint64_t)size) >> 32);
      for (uint32_t step = 0; step < size; ++step) {
        unsigned long long v = a.set_key[at];
        if (v == 0ull) v = atomicCAS(&a.set_key[at], 0ull, (unsigned long long)key);
        if (v == 0ull || v == (unsigned long long)key) break;
        if (++at == size) at = 0u;
      }
      slot = at;
      if (a.set_pos[slot] > p) atomicMin(&a.set_pos[slot], p);
    }
    a.pos_slot[p] = slot;
  }
}

// The batch ends before the first request with a block that an earlier
// request has at another position or behind another block.
__global__ __launch_bounds__(256) void check_kernel(SchedArgs a) {
  __shared__ uint32_t off[kSpecBatch + 1];
  const SchedHdr h = *a.hdr;
  for (uint32_t k = threadIdx.x; k < h.n; k += 256) off[k] = a.off[k];
  __syncthreads();
  const uint32_t stride = gridDim.x * 256u;
  for (uint32_t p = blockIdx.x * 256u + threadIdx.x; p < h.n_pos; p += stride) {
    const uint32_t slot = a.pos_slot[p];
    if (slot == kPosNone) continue;
    const uint32_t f = a.set_pos[slot];
    if (f == p) continue;
    const uint32_t b = batch_of(off, h.n, p), fb = batch_of(off, h.n, f);
    if (fb == b) continue;  // a repeat inside one chain
    const uint32_t j = p - off[b], fj = f - off[fb];
    bool same = j == fj;
    if (same && j > 0u) {
      const ps_req q = a.reqs[h.r0 + b], g = a.reqs[h.r0 + fb];
      same = chain_global(ChainRef{a.pool + q.pre_off, a.pool + q.tail_off, q.pre_len, 0}, (int32_t)j - 1) ==
             chain_global(ChainRef{a.pool + g.pre_off, a.pool + g.tail_off, g.pre_len, 0}, (int32_t)j - 1);
    }
    if (!same && b < a.hdr->stop) atomicMin(&a.hdr->stop, b);
  }
}

// Common prefix of every request with every earlier one, up to the first zero
// hash (equal blocks mean equal prefixes here, so a binary search finds it).
__global__ __launch_bounds__(kSpecBatch) void lcp_kernel(SchedArgs a) {
  const SchedHdr h = *a.hdr;
  const uint32_t b = blockIdx.x, e = threadIdx.x;
  if (b >= h.stop || e >= b) return;
  uint32_t lo = 0u;
  if (a.blen[b] != ~0u && a.blen[e] != ~0u) {
    const ps_req q = a.reqs[h.r0 + b], g = a.reqs[h.r0 + e];
    const ChainRef c{a.pool + q.pre_off, a.pool + q.tail_off, q.pre_len, 0};
    const ChainRef d{a.pool + g.pre_off, a.pool + g.tail_off, g.pre_len, 0};
    uint32_t hi = a.zero_at[b] < a.zero_at[e] ? a.zero_at[b] : a.zero_at[e];
    if (q.pre_off == g.pre_off) {  // one pool segment: equal as far as both go
      lo = (uint32_t)(q.pre_len < g.pre_len ? q.pre_len : g.pre_len);
      lo = lo < hi ? lo : hi;
    }
    while (lo < hi) {  // blocks before lo are equal; position hi differs (or ends)
      const uint32_t mid = (lo + hi) >> 1;
      if (chain_global(c, (int32_t)mid) == chain_global(d, (int32_t)mid)) lo = mid + 1u;
      else hi = mid;
    }
  }
  a.lcp[(size_t)b * kSpecBatch + e] = lo;
}

// ------------------------------------------------ speculative batch scoring
// The kSpecTop least keys a thread has seen, ascending (keys are distinct:
// each ends in its instance id).
struct SpecTop {
  uint64_t k[kSpecTop];
};

__device__ __forceinline__ void spec_push(SpecTop& t, uint64_t key) {
  if (!(key < t.k[kSpecTop - 1])) return;
  t.k[kSpecTop - 1] = key;
#pragma unroll
  for (int j = kSpecTop - 1; j > 0; --j) {
    if (t.k[j] < t.k[j - 1]) {
      const uint64_t x = t.k[j];
      t.k[j] = t.k[j - 1];
      t.k[j - 1] = x;
    }
  }
}

struct SpecShared {
  uint64_t tk[kSpecTop][kSeqMaxThreads];  // each thread's candidates of T, then of C
  uint64_t fk[kSpecTop][kSeqMaxThreads];
  uint64_t red[2][2][kSeqWaves];          // per-wave minima of a merge round (alternating)
  uint32_t cnt[4][kSeqWaves];             // |A|, W_min, |C|, |T| partials
  uint32_t stop[2][2];                    // [round parity][list]: a thread that kept only part
                                          // of its members ran out (read in the next round)
};

// One workgroup per request of a batch (or of a launch of the in-order
// scheduler): Algorithm 1's sets against the
// state at the batch's start (hits from the batch's hits pass), exactly as
// the scheduler evaluates them (same device functions, same fp32 values),
// without a decision: |A|, |C|, |T|, W_min and the first kSpecList members
// of T by the selector's key and of C by the fallback key.  Each thread
// keeps its kSpecTop least keys; the merge takes the least head over the
// threads, one per round, and stops after taking the last kept key of a
// thread that saw more members than it kept (its next member is unknown),
// so every list is the exact start of the ordered set.  Keyed selectors
// only (not Random, not H-C-Q).
__global__ __launch_bounds__(kSeqMaxThreads) void spec_kernel(SpecArgs a) {
  __shared__ SpecShared sh;
  uint32_t r0 = a.r0;
  if (a.hdr) {
    const SchedHdr h = *a.hdr;
    if (blockIdx.x >= h.n) return;
    r0 = h.r0;
  }
  const int tid = threadIdx.x, NT = blockDim.x;
  const int lane = tid & 63, wv = tid >> 6, nwv = NT >> 6;
  const int32_t n_inst = a.n_inst;
  const int32_t r = (int32_t)(r0 + blockIdx.x);
  const ps_req q = a.reqs[r];
  if (!req_valid(q, a.pool_len)) return;  // the scheduler rejects it without a look here
  const DevModel& m = *a.model;
  const ReqLen L{((int64_t)q.pre_len + q.tail_len) * m.bs, q.pre_len + q.tail_len};
  const float Lf = blocks_f(m, L.blocks);
  const float Z = recompute_raw(m, Lf, Lf);
  const float slo = fmaxf(m.ttft_floor, t_prefill(m, Lf, 0.0f));
  const bool kvc = !(m.flags & PS_F_NO_KVC_FILTER) && Z > 0.0f;
  const uint32_t* H = a.hits + (size_t)blockIdx.x * a.stride;
  SpecRec* o = a.out + blockIdx.x;

  // |A| and W_min
  uint32_t al = 0, wl = 0x7F800000u;
  for (int32_t base = 0; base < n_inst; base += kSeqB * NT) {
    InstState st[kSeqB];
    uint32_t hv[kSeqB];
#pragma unroll
    for (int u = 0; u < kSeqB; ++u) {
      const int32_t i = base + u * NT + tid;
      if (i < n_inst) {
        st[u] = a.inst[i];
        hv[u] = H[i];
      }
    }
#pragma unroll
    for (int u = 0; u < kSeqB; ++u) {
      if (base + u * NT + tid >= n_inst || !eligible(m, st[u].A1, st[u].S, L)) continue;
      ++al;
      const uint32_t wb =
          __float_as_uint(fmaxf(0.0f, recompute_raw(m, blocks_f(m, L.blocks - (int32_t)hv[u]), Lf)));
      wl = wb < wl ? wb : wl;
    }
  }
  al = wave_sum_u32(al);
  wl = wave_min_u32(wl);
  if (lane == 0) {
    sh.cnt[0][wv] = al;
    sh.cnt[1][wv] = wl;
  }
  if (tid < 4) sh.stop[tid >> 1][tid & 1] = 0u;
  __syncthreads();
  uint32_t nA = 0, wmin_bits = 0x7F800000u;
  for (int k = 0; k < nwv; ++k) {
    nA += sh.cnt[0][k];
    wmin_bits = sh.cnt[1][k] < wmin_bits ? sh.cnt[1][k] : wmin_bits;
  }
  const float wmin = __uint_as_float(wmin_bits);

  // members of C and T with their keys
  SpecTop tt, ff;
#pragma unroll
  for (int j = 0; j < kSpecTop; ++j) {
    tt.k[j] = ff.k[j] = ~0ull;
  }
  uint32_t cC = 0, cT = 0;
  if (nA > 0) {
    for (int32_t base = 0; base < n_inst; base += kSeqB * NT) {
      InstState st[kSeqB];
      uint32_t hv[kSeqB];
#pragma unroll
      for (int u = 0; u < kSeqB; ++u) {
        const int32_t i = base + u * NT + tid;
        if (i < n_inst) {
          st[u] = a.inst[i];
          hv[u] = H[i];
        }
      }
#pragma unroll
      for (int u = 0; u < kSeqB; ++u) {
        const int32_t i = base + u * NT + tid;
        if (i >= n_inst || !eligible(m, st[u].A1, st[u].S, L)) continue;
        const InstState su = st[u];
        const Member mb = member_with(m, [&]() { return su; }, hv[u], L, Lf, wmin, Z, kvc, slo);
        if (!mb.inC) continue;
        ++cC;
        const uint64_t lm = (uint64_t)(mb.st.P + mb.n_tok) * (uint64_t)mb.st.A1;
        const uint64_t kf =
            (m.flags & PS_F_FALLBACK_DCQ) ? dcq_key(mb.st, hv[u], (uint32_t)i) : ((lm << 16) | (uint32_t)i);
        spec_push(ff, kf);
        if (!mb.inT) continue;
        ++cT;
        spec_push(tt, select_key(m.sel, mb.st, hv[u], (uint32_t)i, lm));
      }
    }
  }
#pragma unroll
  for (int j = 0; j < kSpecTop; ++j) {
    sh.tk[j][tid] = tt.k[j];
    sh.fk[j][tid] = ff.k[j];
  }
  {
    const uint32_t sc = wave_sum_u32(cC), st = wave_sum_u32(cT);
    if (lane == 0) {
      sh.cnt[2][wv] = sc;
      sh.cnt[3][wv] = st;
    }
  }
  __syncthreads();
  uint32_t nC = 0, nT = 0;
  for (int k = 0; k < nwv; ++k) {
    nC += sh.cnt[2][k];
    nT += sh.cnt[3][k];
  }

  // merge: the least heads, one per round
  const int lenT = cT < (uint32_t)kSpecTop ? (int)cT : kSpecTop;
  const int lenF = cC < (uint32_t)kSpecTop ? (int)cC : kSpecTop;
  const bool cutT = cT > (uint32_t)kSpecTop, cutF = cC > (uint32_t)kSpecTop;
  int pT = 0, pF = 0, pb = 0;
  uint32_t nLT = 0, nLF = 0;
  bool doneT = nT == 0u, doneF = nC == 0u;
  for (int round = 0; round < kSpecList && !(doneT && doneF); ++round) {
    const uint64_t hT = (!doneT && pT < lenT) ? sh.tk[pT][tid] : ~0ull;
    const uint64_t hF = (!doneF && pF < lenF) ? sh.fk[pF][tid] : ~0ull;
    const uint64_t mT = wave_min_u64(hT), mF = wave_min_u64(hF);
    if (lane == 0) {
      sh.red[pb][0][wv] = mT;
      sh.red[pb][1][wv] = mF;
    }
    __syncthreads();
    uint64_t gT = ~0ull, gF = ~0ull;
    for (int k = 0; k < nwv; ++k) {
      gT = sh.red[pb][0][k] < gT ? sh.red[pb][0][k] : gT;
      gF = sh.red[pb][1][k] < gF ? sh.red[pb][1][k] : gF;
    }
    pb ^= 1;
    // written in the previous round (each round writes the slot the next
    // one reads, after a barrier that every reader of the slot has passed)
    if (sh.stop[round & 1][0]) doneT = true;
    if (sh.stop[round & 1][1]) doneF = true;
    if (!doneT) {
      if (gT == ~0ull) {
        doneT = true;
      } else {
        if (hT == gT) {
          o->lt[nLT] = gT;
          if (++pT == lenT && cutT) sh.stop[(round + 1) & 1][0] = 1u;
        }
        ++nLT;
      }
    }
    if (!doneF) {
      if (gF == ~0ull) {
        doneF = true;
      } else {
        if (hF == gF) {
          o->lf[nLF] = gF;
          if (++pF == lenF && cutF) sh.stop[(round + 1) & 1][1] = 1u;
        }
        ++nLF;
      }
    }
  }
  if (tid == 0) {
    o->nA = nA;
    o->nC = nC;
    o->nT = nT;
    o->wmin = wmin_bits;
    o->nLT = nLT;
    o->nLF = nLF;
  }
}


// ------------------------------------------------------------------ decisions
// A request's inputs, staged in LDS a request ahead: three parts that a wave
// each fills with one 16-byte load a lane.
struct alignas(16) SchedSlot {
  uint64_t lt[kSpecList], lf[kSpecList];
  uint32_t lcp[kSpecBatch];
  uint32_t head[8];
};
static_assert(kSpecList == 64 && kSpecBatch == 256 && kSeqWaves == 4, "the parts of a slot");
// (LDS, with the dirty bitmap and two staged rows: at most 64 KiB)
struct SchedShared {
  DevModel m;
  SchedSlot slot[2];
  // a request's decision, by request parity: least selector and fallback key
  // and kMoved ... over the changed instances, how many of them were and are in
  // A, C and T (set sizes only); the first listed member of T, or else of C,
  // outside them with its state; barriers beyond the usual ones
  uint64_t kT[2], kF[2];
  uint32_t what[2], cnt[2][6];
  uint64_t t0[2], f0[2];
  InstState st_o[2];
  uint32_t held_o[2];  // its cached blocks
  uint32_t extra[2];
  SeqPart part[2][kSeqWaves];
  uint32_t lmax[2][kSpecBatch];  // per changed instance: longest common prefix with a request on it
  uint32_t u_id[kSpecBatch];     // the changed instances, in order of their first placement
  uint32_t blen[kSpecBatch];
  uint16_t mem[kSpecBatch];      // per request: the changed instance it went to (kNone16: none)
  // the decisions, for the last pass: the chosen instance's state before the
  // placement, its hit now and at the batch's start, flags and set sizes
  InstState st[kSpecBatch];
  int32_t best[kSpecBatch];
  uint32_t hit[kSpecBatch], skip[kSpecBatch], fl[kSpecBatch];
  uint32_t sz[3][kSpecBatch];
  uint32_t scan[kSeqWaves];
  uint32_t stop;
};
static_assert(sizeof(SchedShared) + kSchedRowMax / 8 + 2 * 4 * kSchedRowMax <= 64 * 1024 &&
                  sizeof(SchedShared) + PS_MAX_INST / 8 <= 64 * 1024,
              "LDS of the deciding workgroup");

// Decides the batch in order.  Thread k of the four deciding waves keeps the
// k-th changed instance in registers (its state at the batch's start and
// now); the instances outside are as `spec` saw them.  Per request two steps,
// a barrier after each:
//  E  the deciding waves evaluate every changed instance as it is (as it was,
//     too, for set sizes), with its hit;
//  C  all of them take the decision, and its owner moves the instance's state.
// Five staging waves work beside them: during E four put request b + 1's
// inputs into LDS (loaded during b - 1) and load request b + 2's, and one finds
// the first listed members of T and C outside the changed instances, with the
// state of that instance; during C the four take the longest common prefix of
// request b + 1 with the requests on each changed instance.  So a decision waits for no
// memory, and what bounds it is the deciding waves' own instruction issue (one
// wave, four cycles an instruction) and LDS latency: hence the model in scalar
// registers, ballots instead of reductions, and counts only where asked for.
// 256 decisions on 2,048 instances 656 us, 2.6 us each; with four waves doing
// all of it and three barriers 3.6 us, with memory-waiting barriers and
// generic reductions 4.2 us.
// When a changed instance's hit moved, W_min changed or a list ran out, the
// request is scored over all instances (states and hits only: no table is
// read).
constexpr int kDecideThreads = 2 * kSeqMaxThreads + 64;
__global__ __launch_bounds__(kDecideThreads) void decide_kernel(SchedArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  SchedShared& sh = *reinterpret_cast<SchedShared*>(smem);
  const int32_t n_inst = a.n_inst;
  const uint32_t stride = sched_row_stride(n_inst);
  const int32_t nw = (n_inst + 127) / 128 * 2;
  uint64_t* dirty = reinterpret_cast<uint64_t*>(smem + sizeof(SchedShared));
  uint32_t* rowbuf = reinterpret_cast<uint32_t*>(dirty + nw);  // two rows of hits (row_lds)
  constexpr int NT = kSeqMaxThreads;
  const int lane = threadIdx.x & 63;
  constexpr int nwv = kSeqWaves;
  const SchedHdr h = *a.hdr;
  const uint32_t nb = h.n < h.stop ? h.n : h.stop;
  if (nb == 0u) {
    if (threadIdx.x == 0) *a.commit_hdr = CommitHdr{0u, 0u, 0u, 0u};
    return;
  }
  const bool row_lds = n_inst <= kSchedRowMax;

  auto clear_decision = [&](uint32_t p) {
    sh.kT[p] = sh.kF[p] = ~0ull;
    sh.what[p] = 0u;
    for (int k = 0; k < 6; ++k) sh.cnt[p][k] = 0u;
    sh.extra[p] = 0u;
  };

  if (threadIdx.x >= NT) {  // ------------------------------- the staging waves
    const int tid = threadIdx.x - NT;
    const int wv = (int)uniform_u((uint32_t)tid >> 6);
    // this wave's share of a request's inputs: wave 0 the common prefixes, wave
    // 1 the lists, wave 2 the head (two lanes), and a quarter of the row
    constexpr int kRowVec = kSchedRowMax / 4 / NT;
    uint4 in_part, in_row[kRowVec];
    auto load_inputs = [&](uint32_t b) {
      const SpecRec* sp = a.spec + b;
      const uint4* src = wv == 0   ? reinterpret_cast<const uint4*>(a.lcp + (size_t)b * kSpecBatch) + lane
                         : wv == 1 ? reinterpret_cast<const uint4*>(sp->lt) + lane
                                   : reinterpret_cast<const uint4*>(sp) + (lane & 1);
      in_part = *src;
      if (row_lds) {
        const uint4* r = reinterpret_cast<const uint4*>(a.hits + (size_t)b * stride);
#pragma unroll
        for (int u = 0; u < kRowVec; ++u) in_row[u] = r[4u * (u * NT + tid) < stride ? u * NT + tid : 0];
      }
    };
    auto store_inputs = [&](uint32_t b) {
      SchedSlot& s = sh.slot[b & 1u];
      if (wv == 0) reinterpret_cast<uint4*>(s.lcp)[lane] = in_part;
      else if (wv == 1) reinterpret_cast<uint4*>(s.lt)[lane] = in_part;
      else if (wv == 2 && lane < 2) reinterpret_cast<uint4*>(s.head)[lane] = in_part;
      if (row_lds) {
        uint4* r = reinterpret_cast<uint4*>(rowbuf + (b & 1u) * stride);
#pragma unroll
        for (int u = 0; u < kRowVec; ++u)
          if (4u * (u * NT + tid) < stride) r[u * NT + tid] = in_row[u];
      }
    };
    // a fifth wave looks for the first listed members outside the changed ones
    const bool finder = wv == nwv;
    if (!finder) {
      load_inputs(0u);
      store_inputs(0u);
      load_inputs(nb > 1u ? 1u : 0u);
    }
    __syncthreads();
    for (uint32_t b = 0; b < nb; ++b) {
      const uint32_t p = b & 1u;
      const SchedSlot& in = sh.slot[p];
      const bool valid = sh.blen[b] != ~0u;
      // E
      if (finder && valid) {
        const uint32_t s_nLT = uniform_u(in.head[4]), s_nLF = uniform_u(in.head[5]);
        const uint64_t t0 = spec_first_outside(in.lt[lane], s_nLT, dirty, lane);
        const uint64_t f0 = t0 == ~0ull ? spec_first_outside(in.lf[lane], s_nLF, dirty, lane) : ~0ull;
        const uint64_t o0 = t0 != ~0ull ? t0 : f0;
        InstState st{};
        uint32_t held = 0u;
        if (o0 != ~0ull) {
          st = a.inst[o0 & 0xFFFFu];
          held = a.t.count[o0 & 0xFFFFu];
        }
        if (lane == 0) {
          sh.t0[p] = t0;
          sh.f0[p] = f0;
          sh.st_o[p] = st;
          sh.held_o[p] = held;
        }
      }
      // (slot and row b + 1 were last read before the barrier that ended b - 1)
      if (!finder) {
        store_inputs(b + 1u);
        load_inputs(b + 2u < nb ? b + 2u : nb - 1u);
      }
      lds_barrier();
      // C: request b + 1's common prefixes with the requests before b (b's
      // owner adds b's); request b's are read
      if (!finder) {
        sh.lmax[p][tid] = 0u;
        if ((uint32_t)tid < b && sh.mem[tid] != kNone16)
          atomicMax(&sh.lmax[p ^ 1u][sh.mem[tid]], sh.slot[p ^ 1u].lcp[tid]);
      } else if (lane == 0) {
        clear_decision(p ^ 1u);  // last read before this request
      }
      lds_barrier();
      // barriers beyond these: the first of them was the one just passed
      const uint32_t extra = uniform_u(sh.extra[p]);
      if (extra && uniform_u(sh.stop)) {
        __syncthreads();
        break;
      }
      for (uint32_t k = 0; k < extra; ++k) lds_barrier();
    }
    for (int k = 0; k < 4; ++k) __syncthreads();  // the deciding waves' last passes
    return;
  }

  // --------------------------------------------------------- the deciding waves
  const int tid = threadIdx.x;
  const int wv = (int)uniform_u((uint32_t)tid >> 6);
  stage_model(sh.m, a.model, tid, NT);
  for (int32_t w = tid; w < nw; w += NT) dirty[w] = 0ull;
  sh.blen[tid] = a.blen[tid];
  sh.mem[tid] = (uint16_t)kNone16;
  sh.lmax[0][tid] = sh.lmax[1][tid] = 0u;
  if (tid == 0) {
    sh.stop = 0u;
    clear_decision(0u);
    clear_decision(1u);
  }
  // the k-th changed instance of this thread
  uint32_t u_my = ~0u, room_my = 0u, cnt_my = 0u;  // room: blocks its cap leaves; cnt: new ones, at most
  InstState so{}, sc{};
  uint32_t n_u = 0u, done = nb, n_fast = 0u, n_full = 0u;
  int pb = 0;
  __syncthreads();
  const ModelRegs m = model_regs(sh.m);
  const int32_t ub_lane = lane < m.n_seg ? m.seg_ub[lane] : INT32_MAX;  // ascending
  const bool want_sizes = a.sizes != nullptr;

  for (uint32_t b = 0; b < nb; ++b) {
    const uint32_t p = b & 1u;
    const SchedSlot& in = sh.slot[p];
    uint32_t* hl = rowbuf + (row_lds ? p * stride : 0u);
    uint32_t* hg = a.hits + (size_t)b * stride;
    // (two branches, so that neither is a flat access)
    auto hit_of = [&](uint32_t i) -> uint32_t {
      if (row_lds) return hl[i];
      return hg[i];
    };
    const uint32_t len = uniform_u(sh.blen[b]);
    const uint32_t wmin_b = uniform_u(in.head[3]);
    const bool valid = len != ~0u;
    const int32_t ell = valid ? (int32_t)len : 0;
    const ReqLen L{(int64_t)ell * m.bs, ell};
    const float Lf = blocks_f(m, L.blocks);
    int32_t best = -1;
    uint32_t fl = valid ? PS_R_REJECT : PS_R_INVALID, nA = 0, nC = 0, nT = 0;
    bool outside = false;  // the choice is not a changed instance
    bool full = false;     // scored over all instances
    uint32_t h_my = 0u, hx_my = 0u;
    InstState st_full{};
    uint32_t held_full = 0u;
    if (!valid) lds_barrier();
    if (valid) {
      const float Z = recompute_raw(m, Lf, Lf);  // T_pf(L, 0) - T_pf(0, L)
      const float slo = fmaxf(m.ttft_floor, t_prefill(m, Lf, 0.0f));
      const bool kvc = !(m.flags & PS_F_NO_KVC_FILTER) && Z > 0.0f;
      const float wmin = __uint_as_float(wmin_b);
      // E
      const bool mine = (uint32_t)tid < n_u;
      uint64_t keyT = ~0ull, keyF = ~0ull;
      if ((uint32_t)(wv * 64) < n_u) {
        bool eb = false, ec = false, cb = false, cc = false, tb = false, tc = false;
        uint32_t wb = ~0u;
        if (mine) {
          // (an instance at its cap takes no blocks, so its hits stay)
          const uint32_t lm = room_my ? sh.lmax[p][tid] : 0u;
          h_my = hit_of(u_my);
          hx_my = lm > h_my ? lm : h_my;
          eb = eligible(m, so.A1, so.S, L);
          ec = eligible(m, sc.A1, sc.S, L);
          wb = __float_as_uint(fmaxf(0.0f, recompute_raw(m, blocks_f(m, L.blocks - (int32_t)h_my), Lf)));
          if (want_sizes && eb) {
            const Member mb = member_with(m, [&]() { return so; }, h_my, L, Lf, wmin, Z, kvc, slo);
            cb = mb.inC;
            tb = mb.inT;
          }
          if (ec) {
            const Member mb = member_with(m, [&]() { return sc; }, h_my, L, Lf, wmin, Z, kvc, slo);
            if (mb.inC) {
              cc = true;
              const uint64_t lmk = (uint64_t)(mb.st.P + mb.n_tok) * (uint64_t)mb.st.A1;
              keyF = (m.flags & PS_F_FALLBACK_DCQ) ? dcq_key(mb.st, h_my, u_my) : ((lmk << 16) | u_my);
              if (mb.inT) {
                tc = true;
                keyT = select_key(m.sel, mb.st, h_my, u_my, lmk);
              }
            }
          }
        }
        const uint32_t what =
            (__ballot(ec && hx_my > h_my) ? kMoved : 0u) | (__ballot(ec && wb < wmin_b) ? kBelow : 0u) |
            (__ballot(eb && wb == wmin_b) ? kMinThen : 0u) | (__ballot(ec && wb == wmin_b) ? kMinNow : 0u);
        const uint64_t btc = __ballot(tc);
        if (btc) {
          const uint64_t k = wave_min_u64(keyT);
          if (lane == 0) atomicMin(reinterpret_cast<unsigned long long*>(&sh.kT[p]), (unsigned long long)k);
        }
        if (what && lane == 0) atomicOr(&sh.what[p], what);
        if (want_sizes) {
          const uint32_t n[6] = {(uint32_t)__popcll(__ballot(eb)), (uint32_t)__popcll(__ballot(ec)),
                                 (uint32_t)__popcll(__ballot(cb)), (uint32_t)__popcll(__ballot(cc)),
                                 (uint32_t)__popcll(__ballot(tb)), (uint32_t)__popcll(btc)};
          if (lane == 0)
            for (int k = 0; k < 6; ++k)
              if (n[k]) atomicAdd(&sh.cnt[p][k], n[k]);
        }
      }
      lds_barrier();
      // C
      const uint32_t s_nC = uniform_u(in.head[1]), s_nT = uniform_u(in.head[2]), s_nLT = uniform_u(in.head[4]),
                     s_nLF = uniform_u(in.head[5]);
      const uint64_t t0 = sh.t0[p], kTm = sh.kT[p];
      const uint32_t what = sh.what[p];
      const uint64_t kT = t0 < kTm ? t0 : kTm;
      // W_min is unchanged unless a hit moved, or the only changed instances
      // at the minimum all left A: then it is not known here.  The other
      // members of T and C are as speculated; the first listed one outside is
      // the least of them when the list shows it.
      bool ok = uniform_u(!(what & (kMoved | kBelow)) && (what & (kMinThen | kMinNow)) != kMinThen &&
                          !(t0 == ~0ull && s_nLT < s_nT)) != 0u;
      const bool some = uniform_u(kT != ~0ull) != 0u;
      if (ok && some) {
        best = (int32_t)uniform_u((uint32_t)kT & 0xFFFFu);
        fl = 0;
        outside = uniform_u(t0 < kTm) != 0u;
      } else if (ok) {  // T is empty: the fallback keys
        const uint64_t f0 = sh.f0[p];
        if (uniform_u(f0 == ~0ull) && s_nLF < s_nC) {
          ok = false;
        } else {
          if ((uint32_t)(wv * 64) < n_u) {
            const uint64_t k = wave_min_u64(keyF);
            if (lane == 0) atomicMin(reinterpret_cast<unsigned long long*>(&sh.kF[p]), (unsigned long long)k);
          }
          if (tid == 0) sh.extra[p] = 1u;
          lds_barrier();
          const uint64_t kFm = sh.kF[p];
          const uint64_t kF = f0 < kFm ? f0 : kFm;
          if (uniform_u(kF != ~0ull)) {
            best = (int32_t)uniform_u((uint32_t)kF & 0xFFFFu);
            fl = PS_R_FALLBACK;
            outside = uniform_u(f0 < kFm) != 0u;
          }
        }
      }
      if (ok) {
        ++n_fast;
        if (want_sizes) {
          nA = in.head[0] - sh.cnt[p][0] + sh.cnt[p][1];
          nC = s_nC - sh.cnt[p][2] + sh.cnt[p][3];
          nT = s_nT - sh.cnt[p][4] + sh.cnt[p][5];
        }
      } else {
        full = true;
        // every instance: the changed ones' hits moved on to the common
        // prefix, unless the table goes on there or its cap may have refused
        // blocks of it: then the batch ends before this request
        if (tid == 0) sh.extra[p] = 5u;
        if (mine && hx_my > h_my && eligible(m, sc.A1, sc.S, L)) {
          bool bad = cnt_my > room_my;
          if (!bad && (int32_t)hx_my < ell) {
            const ps_req q = a.reqs[h.r0 + b];
            bad = probe(a.t, u_my, chain_global(ChainRef{a.pool + q.pre_off, a.pool + q.tail_off, q.pre_len, ell},
                                                (int32_t)hx_my));
          }
          if (bad) sh.stop = 1u;
        }
        __syncthreads();
        if (mine) {
          a.inst[u_my] = sc;  // read below by every wave
          if (row_lds) hl[u_my] = hx_my;
          else hg[u_my] = hx_my;
        }
        __syncthreads();
        if (uniform_u(sh.stop)) {
          done = b;
          break;
        }
        ++n_full;
        uint32_t al = 0, wl = 0x7F800000u;
        for (int32_t base = 0; base < n_inst; base += NT) {
          const int32_t i = base + tid;
          if (i >= n_inst) continue;
          const InstState st = a.inst[i];
          if (!eligible(m, st.A1, st.S, L)) continue;
          ++al;
          const uint32_t wb =
              __float_as_uint(fmaxf(0.0f, recompute_raw(m, blocks_f(m, L.blocks - (int32_t)hit_of((uint32_t)i)), Lf)));
          wl = wb < wl ? wb : wl;
        }
        al = wave_sum_u32(al);
        wl = wave_min_u32(wl);
        if (lane == 0) {
          sh.part[pb][wv].nA = al;
          sh.part[pb][wv].wmin = wl;
        }
        lds_barrier();
        uint32_t wmin_bits = 0x7F800000u;
        for (int k = 0; k < nwv; ++k) {
          nA += sh.part[pb][k].nA;
          wmin_bits = sh.part[pb][k].wmin < wmin_bits ? sh.part[pb][k].wmin : wmin_bits;
        }
        pb ^= 1;
        const float wm = __uint_as_float(wmin_bits);
        Acc acc{~0ull, ~0ull, ~0u, 0u, 0u};
        for (int32_t base = 0; base < n_inst; base += NT) {
          const int32_t i = base + tid;
          if (i >= n_inst) continue;
          const InstState st = a.inst[i];
          if (!eligible(m, st.A1, st.S, L)) continue;
          evaluate_with(m, acc, (uint32_t)i, hit_of((uint32_t)i), [&]() { return st; }, L, Lf, wm, Z, kvc, slo);
        }
        const uint64_t kTw = wave_min_u64(acc.keyT), kFw = wave_min_u64(acc.keyF);
        const uint32_t cC = wave_sum_u32(acc.nC), cT = wave_sum_u32(acc.nT);
        if (lane == 0) {
          SeqPart& sp = sh.part[pb][wv];
          sp.keyT = kTw;
          sp.keyF = kFw;
          sp.nC = cC;
          sp.nT = cT;
        }
        lds_barrier();
        uint64_t gT = ~0ull, gF = ~0ull;
        for (int k = 0; k < nwv; ++k) {
          const SeqPart& sp = sh.part[pb][k];
          gT = sp.keyT < gT ? sp.keyT : gT;
          gF = sp.keyF < gF ? sp.keyF : gF;
          nC += sp.nC;
          nT += sp.nT;
        }
        pb ^= 1;
        if (uniform_u(gT != ~0ull || gF != ~0ull)) {
          fl = uniform_u(gT != ~0ull) ? 0u : PS_R_FALLBACK;
          best = (int32_t)(uniform_u((uint32_t)(gT != ~0ull ? gT : gF)) & 0xFFFFu);
          outside = uniform_u(!test_bit(dirty, (uint32_t)best)) != 0u;
          if (outside) {
            st_full = a.inst[best];
            held_full = a.t.count[best];
          }
        }
        lds_barrier();  // `outside` read before the owner marks the instance
      }
    }
    if (best < 0) {
      if (tid == 0) {
        sh.best[b] = -1;
        sh.fl[b] = fl;
      }
    } else {
      // the owner's wave: the segment of the batch size after the placement
      // from a ballot over the bounds
      const uint64_t om = outside ? ((uint32_t)wv == n_u >> 6 ? 1ull << (n_u & 63u) : 0ull)
                                  : __ballot((uint32_t)tid < n_u && u_my == (uint32_t)best);
      if (om) {
        const int ol = __builtin_ctzll(om);
        if (outside && lane == ol) {
          u_my = (uint32_t)best;
          so = sc = full ? st_full : sh.st_o[p];
          cnt_my = 0u;
          const uint32_t held = full ? held_full : sh.held_o[p];
          room_my = a.cap > held ? a.cap - held : 0u;
          h_my = hit_of((uint32_t)best);
          hx_my = h_my;
          sh.u_id[n_u] = u_my;
          dirty[best >> 6] |= 1ull << (best & 63);
        }
        const int32_t a1 = __builtin_amdgcn_readlane(sc.A1, ol) + 1;
        const int32_t seg = (int32_t)__popcll(__ballot(ub_lane < a1));  // lanes past the segments never count
        if (lane == ol) {
          const uint32_t v = hx_my;
          sh.mem[b] = (uint16_t)tid;
          atomicMax(&sh.lmax[p ^ 1u][tid], sh.slot[p ^ 1u].lcp[b]);
          sh.best[b] = best;
          sh.st[b] = sc;
          sh.hit[b] = v;
          sh.skip[b] = h_my;
          sh.fl[b] = fl;
          sc.Q += 1;
          sc.A1 = a1;
          sc.P += L - (int64_t)v * m.bs;
          sc.S += L;
          sc.seg = seg < m.n_seg ? seg : m.n_seg - 1;
          cnt_my += (uint32_t)ell - v;
        }
      }
      if (outside) ++n_u;
    }
    if (want_sizes && tid == 0) {
      sh.sz[0][b] = nA;
      sh.sz[1][b] = nC;
      sh.sz[2][b] = nT;
    }
    lds_barrier();
  }
  // the changed instances' states
  if ((uint32_t)tid < n_u) {
    a.inst[u_my] = sc;
    a.room[u_my] = sc.A1 <= m.b_max ? m.kv_cap - sc.S : -1;
  }
  __syncthreads();

  // Results: a thread per request.
  const uint32_t t = (uint32_t)tid;
  if (t < done) {
    const uint32_t r = h.r0 + t;
    const int32_t best = sh.best[t];
    uint32_t fl = sh.fl[t];
    if (best < 0) {
      a.out[r] = ps_result{-1, 0, 0.0f, 0.0f, fl};
    } else {
      const ReqLen L{(int64_t)sh.blen[t] * m.bs, (int32_t)sh.blen[t]};
      const InstState st = sh.st[t];
      const Lat lt = latency(m, st, blocks_f(m, L.blocks - (int32_t)sh.hit[t]), blocks_f(m, (int32_t)sh.hit[t]), L);
      if (lt.ttft > fmaxf(m.ttft_floor, t_prefill(m, blocks_f(m, L.blocks), 0.0f))) fl |= PS_R_TTFT_MISS;
      a.out[r] = ps_result{best, (int32_t)sh.hit[t], lt.ttft, lt.tpot, fl};
    }
    if (a.sizes) {
      const bool inv = (fl & PS_R_INVALID) != 0u;
      for (int k = 0; k < 3; ++k) a.sizes[3 * (size_t)r + k] = inv ? 0u : sh.sz[k][t];
    }
  }

  // The commit batch: the placed requests grouped by instance, arrival order
  // inside a group (thread k: the k-th changed instance).
  uint32_t n_my = 0u;
  if (t < n_u)
    for (uint32_t e = 0; e < done; ++e) n_my += sh.mem[e] == t ? 1u : 0u;
  uint32_t e0 = wave_exclusive_sum(n_my, lane);
  if (lane == 63) sh.scan[wv] = e0 + n_my;
  __syncthreads();
  uint32_t n_ent = 0u;
  for (int k = 0; k < nwv; ++k) {
    if (k < wv) e0 += sh.scan[k];
    n_ent += sh.scan[k];
  }
  uint32_t len_my = 0u;
  if (t < n_u) {
    a.grp_inst[t] = (int32_t)sh.u_id[t];
    a.grp_ent[t] = e0;
    uint32_t at = e0;
    for (uint32_t e = 0; e < done; ++e) {
      if (sh.mem[e] != t) continue;
      a.ent_req[at] = (int32_t)(h.r0 + e);
      a.ent_grp[at] = t;
      a.ent_skip[at] = sh.skip[e];
      ++at;
      len_my += sh.blen[e];
    }
  }
  __syncthreads();
  uint32_t p0 = wave_exclusive_sum(len_my, lane);
  if (lane == 63) sh.scan[wv] = p0 + len_my;
  __syncthreads();
  uint32_t n_pos = 0u;
  for (int k = 0; k < nwv; ++k) {
    if (k < wv) p0 += sh.scan[k];
    n_pos += sh.scan[k];
  }
  if (t < n_u) {
    uint32_t at = e0;
    for (uint32_t e = 0; e < done; ++e) {
      if (sh.mem[e] != t) continue;
      a.ent_off[at++] = p0;
      p0 += sh.blen[e];
    }
  }
  if (tid == 0) {
    a.grp_ent[n_u] = n_ent;
    a.ent_off[n_ent] = n_pos;
    *a.commit_hdr = CommitHdr{n_ent, n_u, n_pos, 0u};
    *a.cursor = h.r0 + done;
    atomicAdd(a.stats, (unsigned long long)n_fast);
    atomicAdd(a.stats + 1, (unsigned long long)n_full);
  }
}

}  // namespace

hipError_t ps_launch_spec(const SpecArgs& a, uint32_t n, hipStream_t s) {
  if (n == 0u) return hipSuccess;
  hipLaunchKernelGGL(spec_kernel, dim3(n), dim3(kSeqMaxThreads), 0, s, a);
  return hipGetLastError();
}

size_t ps_sched_lds_bytes(int32_t n_inst) {
  return sizeof(SchedShared) + ((size_t)n_inst + 127) / 128 * 2 * sizeof(uint64_t) +
         (n_inst <= kSchedRowMax ? 2 * (size_t)sched_row_stride(n_inst) * sizeof(uint32_t) : 0);
}

hipError_t ps_launch_sched_batch(const SchedArgs& a, hipStream_t s) {
  const unsigned n = a.max_n;
  const unsigned pgrid = std::min(std::max((a.max_pos + 255u) / 256u, 1u), 4096u);
  hipLaunchKernelGGL(plan_kernel, dim3(1), dim3(kSpecBatch), 0, s, a);
  hipLaunchKernelGGL(first_kernel, dim3(n, std::min(((unsigned)a.n_inst + 255u) / 256u, 256u)), dim3(256), 0, s, a);
  hipLaunchKernelGGL(walk_kernel, dim3(4096), dim3(64), 0, s, a);
  const SpecArgs sa{a.hdr, 0u, a.inst, a.model, a.reqs, a.pool_len, a.n_inst, a.hits, sched_row_stride(a.n_inst),
                    a.spec};
  hipLaunchKernelGGL(spec_kernel, dim3(n), dim3(kSeqMaxThreads), 0, s, sa);
  hipLaunchKernelGGL(intern_clear_kernel, dim3(pgrid), dim3(256), 0, s, a);
  hipLaunchKernelGGL(intern_kernel, dim3(pgrid), dim3(256), 0, s, a);
  hipLaunchKernelGGL(check_kernel, dim3(pgrid), dim3(256), 0, s, a);
  hipLaunchKernelGGL(lcp_kernel, dim3(n), dim3(kSpecBatch), 0, s, a);
  hipLaunchKernelGGL(decide_kernel, dim3(1), dim3(kDecideThreads), ps_sched_lds_bytes(a.n_inst), s, a);
  return hipGetLastError();
}
