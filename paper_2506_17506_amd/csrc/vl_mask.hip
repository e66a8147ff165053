// Constrained-decoding mask (Section 4.5, last sentence of the error analysis: mask out the
// registers that are occupied while the allocation is generated): for the occurrence a
// decoder has reached, the bases that keep consistency, realizability and safety
// (Section 3.4) intact against the occurrences already emitted.  P(i) is rebuilt from the
// analysis' event stream the way the verifier's pair search does.
//
// The samples of one kernel reach an occurrence together, and their rows usually lie at equal
// distances: the host folds such neighbouring queries into runs (program, occurrence, first row,
// distance, count), and a workgroup rebuilds P(i) once for its share of a run; then a wavefront
// answers a query at a time.  What bounds a call is waiting: some eight dependent reads
// (one program x 100: 5.9 us; 12.2 when every lane looked up the members of its bitset words one after the other), and on the host the pass over the queries.  A workgroup per query, each with a
// table entry to upload, took 28 us on the device and 51 us in all for 6,400 queries.
#include <algorithm>
#include <cstring>
#include <mutex>
#include <type_traits>

#include "vl_dev.h"

using namespace vl;

namespace {

struct Run {
  const DevMir *mir;
  const DevLive *live;
  const uint16_t *cand;   // row of the first query; query x reads from cand + x * stride
  int64_t stride;
  uint32_t occ, count, first_query, first_block;
};
constexpr uint32_t kArgRuns = 64;   // runs that travel as a kernel argument (3 KB); more go through a table, whose upload costs 7 us
                                   // (runs of 20 queries: 64 take 12.3 us, 65 19.2)
struct RunArgs { Run run[kArgRuns]; };
constexpr uint32_t kMaskThreads = 256, kMaskWaves = kMaskThreads / 64;
// members of P(i) that are listed: those in the way, and all where they are found by their bits (in the same memory,
// before that); with more, every vreg gets a turn
constexpr uint32_t kMaskMembers = 256, kMaskListed = 2 * kMaskMembers;

template <bool kByArgument>
__global__ __launch_bounds__(kMaskThreads) void k_free_bases(const std::conditional_t<kByArgument, RunArgs, const Run *> args, uint32_t n_runs,
                                                             uint32_t per_block, uint32_t *__restrict__ masks) {
  const Run *runs;
  if constexpr (kByArgument) runs = args.run;
  else runs = args;
  const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
  // the run of this block: 64 probes at a time, one per lane
  uint32_t at = 0, len = n_runs;
  while (len > 1) {
    const uint32_t step = (len + 63u) / 64u, off = lane * step;
    const uint32_t n = (uint32_t)__popcll(__ballot(off < len && runs[at + off].first_block <= blockIdx.x));
    at += (n - 1u) * step;
    len = min(step, len - (n - 1u) * step);
  }
  const Run R = runs[at];
  const DevMir VL_GLOBAL &m = *as_global(R.mir);
  const DevLive VL_GLOBAL &L = *as_global(R.live);
  extern __shared__ uint32_t in_p[];                  // [W] members of P(i)
  __shared__ uint2 members[kMaskMembers];             // (first occurrence, width) of those in the way
  __shared__ uint32_t n_members;
  __shared__ uint32_t n_listed;
  __shared__ uint32_t blocked_all[kMaskWaves][17];    // registers that are taken or reserved (word 16: always zero)
  uint32_t *const blocked = blocked_all[wave];
  const uint32_t q = R.occ, v = m.occ_vreg[q], i = m.occ_instr[q];
  const uint32_t attr = m.vattr[v], cls = attr_class(attr), width = attr_width(attr), align = attr_align(attr);
  const uint32_t F = m.class_size[cls];
  const uint32_t first_v = L.first[v];
  const bool fresh = first_v >= q;   // the first mention of v: everything in P(i) that already has a register is in the way
  auto in_the_way = [&](uint32_t b, uint2 &out) {
    const uint32_t ab = m.vattr[b], fb = L.first[b];
    out = make_uint2(fb, attr_width(ab));
    return b != v && attr_class(ab) == cls && fb < q;
  };
  bool listed_once = false;   // what is in `members` has no bit any more
  if (fresh) {
    for (uint32_t x = threadIdx.x; x < m.W; x += kMaskThreads) in_p[x] = 0;
    if (threadIdx.x == 0) n_members = n_listed = 0;
    // Short lists: the records are kept until the bits say which of them are members.  A record
    // has its value's width and class, so that only the first occurrence is looked up, all of a thread's at once.
    // Longer ones: the members are listed from the bits, and looked up a lane each.  (4,000 instructions in one tile, one
    // program x 100 and 64 x 100: 9.6 and 23 us; 14.5 and 30 when the records beyond those kept were read one at a time, twice.)
    const RecordsOfP p = records_of_p(m, L, i);
    KeptRecords<1, 3, kMaskThreads> kept;
    const bool fit = listed_once = kept.fit(p);
    if (fit) kept.load(L, p, threadIdx.x);
    __syncthreads();
    if (fit) kept.flip(in_p);
    else flip_members_of_p(L, p, in_p, threadIdx.x, kMaskThreads);
    __syncthreads();
    auto list = [&](uint2 e) {
      const uint32_t slot = atomicAdd(&n_members, 1u);
      if (slot < kMaskMembers) members[slot] = e;
      return slot < kMaskMembers;
    };
    if (fit) {
      uint32_t fb[kept.kAll];
#pragma unroll
      for (uint32_t u = 0; u < kept.kAll; ++u) {   // members of v's class (classes begin at different mask words) other than v
        const u32x4 r = kept.rec[u];
        const uint32_t b = r.x >> 8;
        fb[u] = kNone;
        if (r.y && b != v && r.z == attr_word(attr) * 256u && is_member(in_p, b)) fb[u] = L.first[b];
      }
#pragma unroll
      for (uint32_t u = 0; u < kept.kAll; ++u) {
        if (fb[u] >= q) continue;
        // A value may have several records: the one that finds its bit lists it, and takes the bit.  (As many entries as
        // records: 30 values written four times in a tile of 512, one program x 100:
        // 19.7 us a launch, since every vreg then has its turn; 5.5 this way.)
        const uint32_t b = kept.rec[u].x >> 8, bit = 1u << (b & 31);
        if (!(__hip_atomic_fetch_and(&in_p[b >> 5], ~bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) & bit)) continue;
        if (!list(make_uint2(fb[u], (uint32_t)__popc(kept.rec[u].y)))) atomicOr(&in_p[b >> 5], bit);   // no room: found by its bit
      }
    } else {
      uint32_t *const listed = &members[0].x;
      list_members(in_p, m.W, listed, kMaskListed, &n_listed, threadIdx.x, kMaskThreads);
      __syncthreads();
      constexpr uint32_t kEach = kMaskListed / kMaskThreads;
      uint2 mine[kEach];
      bool taken[kEach];
#pragma unroll
      for (uint32_t u = 0; u < kEach; ++u) {
        const uint32_t y = threadIdx.x + u * kMaskThreads;
        taken[u] = y < n_listed && in_the_way(listed[y], mine[u]);
      }
      __syncthreads();
#pragma unroll
      for (uint32_t u = 0; u < kEach; ++u)
        if (taken[u]) list(mine[u]);
      if (threadIdx.x == 0 && n_listed > kMaskListed) atomicAdd(&n_members, kMaskMembers + 1u);   // every vreg gets a turn
    }
    __syncthreads();
  }
  const uint32_t wm = width == 32 ? 0xFFFFFFFFu : ((1u << width) - 1u);
  const uint32_t x0 = (blockIdx.x - R.first_block) * per_block, x1 = min(R.count, x0 + per_block);
  for (uint32_t x = x0 + wave; x < x1; x += kMaskWaves) {
    const uint16_t VL_GLOBAL *row = as_global(R.cand) + (int64_t)x * R.stride;
    if (lane < 17) blocked[lane] = (lane < 16 && m.has_reserved) ? m.reserved[cls][lane] : 0u;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    auto take = [&](uint2 e) {
      const uint32_t p = row[e.x];
      for (uint32_t r = p; r < p + e.y && r < 512u; r = (r | 31u) + 1u) {   // one word after the other
        const uint32_t n = min(p + e.y - r, 32u - (r & 31u));
        atomicOr(&blocked[r >> 5], (n == 32u ? 0xFFFFFFFFu : ((1u << n) - 1u)) << (r & 31u));
      }
    };
    if (fresh) {
      const bool all = n_members <= kMaskMembers;
      if (all || listed_once)
        for (uint32_t y = lane; y < min(n_members, kMaskMembers); y += 64) take(members[y]);
      if (!all) {
        for (uint32_t b = lane; b < m.V; b += 64) {
          uint2 e;
          if (is_member(in_p, b) && in_the_way(b, e)) take(e);
        }
      }
    }
    const uint32_t forced = fresh ? kNone : (uint32_t)row[first_v];   // a later mention: only its own register
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    // 64 consecutive bases per turn: two words of the mask, which end up in lanes 0 .. 15
    uint32_t mine = 0;
#pragma unroll
    for (uint32_t t = 0; t < 8; ++t) {
      const uint32_t p = t * 64u + lane;
      const uint64_t window = ((uint64_t)blocked[p >> 5] | ((uint64_t)blocked[(p >> 5) + 1] << 32)) >> (p & 31);
      bool ok = p % align == 0 && p + width <= F && ((uint32_t)window & wm) == 0;
      if (forced != kNone && p != forced) ok = false;
      const uint64_t ballot = __ballot(ok);
      if (lane >> 1 == t) mine = (lane & 1u) ? (uint32_t)(ballot >> 32) : (uint32_t)ballot;
    }
    if (lane < 16) masks[(size_t)(R.first_query + x) * 16 + lane] = mine;
    __builtin_amdgcn_wave_barrier();   // the wavefront's words are rewritten by its next query
  }
}

// Runs of a query or two, a workgroup each: nothing to share out, so two wavefronts do everything
// together.  The members of P(i) are first listed, which takes no reads from memory, and then looked up a lane
// each.  (us per call, a workgroup of four wavefronts for each of them / this: 1,000 scattered queries of a program of
// 8,000 instructions 31 / 25, 4,000 42 / 30, 16,000 121 / 56; of first mentions 31 / 25, 55 / 32, 153 / 66;
// 29, 35, 63 and 30, 38, 81 with a workgroup of two that looked every vreg up.)
constexpr uint32_t kAloneThreads = 128, kAloneMembers = 512;   // (members that are listed; with more, every vreg gets a turn)
__global__ __launch_bounds__(kAloneThreads) void k_free_bases_alone(const Run *__restrict__ runs, uint32_t *__restrict__ masks) {
  const Run R = runs[blockIdx.x];
  const DevMir VL_GLOBAL &m = *as_global(R.mir);
  const DevLive VL_GLOBAL &L = *as_global(R.live);
  extern __shared__ uint32_t in_p[];      // [W] members of P(i)
  __shared__ uint32_t members[kAloneMembers], n_members;
  __shared__ uint32_t blocked[17];        // registers that are taken or reserved (word 16: always zero)
  const uint32_t tid = threadIdx.x, q = R.occ, v = m.occ_vreg[q], i = m.occ_instr[q];
  const uint32_t attr = m.vattr[v], cls = attr_class(attr), width = attr_width(attr), align = attr_align(attr);
  const uint32_t F = m.class_size[cls], first_v = L.first[v];
  const bool fresh = first_v >= q;   // the first mention of v: everything in P(i) that already has a register is in the way
  if (fresh) {
    for (uint32_t x = tid; x < m.W; x += kAloneThreads) in_p[x] = 0;
    if (tid == 0) n_members = 0;
    __syncthreads();
    flip_members_of_p(L, records_of_p(m, L, i), in_p, tid, kAloneThreads);
    __syncthreads();
    list_members(in_p, m.W, members, kAloneMembers, &n_members, tid, kAloneThreads);
  }
  const uint32_t wm = width == 32 ? 0xFFFFFFFFu : ((1u << width) - 1u);
  for (uint32_t x = 0; x < R.count; ++x) {
    const uint16_t VL_GLOBAL *row = as_global(R.cand) + (int64_t)x * R.stride;
    if (tid < 17) blocked[tid] = (tid < 16 && m.has_reserved) ? m.reserved[cls][tid] : 0u;
    __syncthreads();
    auto take = [&](uint32_t b) {
      const uint32_t ab = m.vattr[b], fb = L.first[b];
      if (b == v || attr_class(ab) != cls || fb >= q) return;
      const uint32_t p = row[fb], end = p + attr_width(ab);
      for (uint32_t r = p; r < end && r < 512u; r = (r | 31u) + 1u) {   // one word after the other
        const uint32_t n = min(end - r, 32u - (r & 31u));
        atomicOr(&blocked[r >> 5], (n == 32u ? 0xFFFFFFFFu : ((1u << n) - 1u)) << (r & 31u));
      }
    };
    if (fresh) {
      if (n_members <= kAloneMembers) {
        for (uint32_t y = tid; y < n_members; y += kAloneThreads) take(members[y]);
      } else {
        for (uint32_t b = tid; b < m.V; b += kAloneThreads)
          if (is_member(in_p, b)) take(b);
      }
      __syncthreads();
    }
    const uint32_t forced = fresh ? kNone : (uint32_t)row[first_v];   // a later mention: only its own register
    uint32_t *const out = masks + (size_t)(R.first_query + x) * 16;
#pragma unroll
    for (uint32_t p = tid; p < 512u; p += kAloneThreads) {
      const uint64_t window = ((uint64_t)blocked[p >> 5] | ((uint64_t)blocked[(p >> 5) + 1] << 32)) >> (p & 31);
      bool ok = p % align == 0 && p + width <= F && ((uint32_t)window & wm) == 0;
      if (forced != kNone && p != forced) ok = false;
      const uint64_t ballot = __ballot(ok);   // a wavefront covers 64 consecutive bases: two words of the mask
      if ((tid & 63u) < 2u) out[(p >> 6) * 2u + (tid & 1u)] = (tid & 1u) ? (uint32_t)(ballot >> 32) : (uint32_t)ballot;
    }
    __syncthreads();   // the words are rewritten by the next query
  }
}

// tables of runs on the device, one set per device, for calls with more runs than fit the kernel's
// argument; used in turn, so that a call waits only for the one kTables calls ago
constexpr uint32_t kTables = 4, kLeastRuns = 4096;
struct Tables {
  std::mutex mu;
  struct One {
    Run *dev = nullptr, *host = nullptr;   // host: pinned
    uint32_t cap = 0, dev_cap = 0;         // runs there is room for in host, in dev
    hipEvent_t consumed = nullptr;         // recorded after the kernel that reads the table
    bool in_flight = false;
  } one[kTables];
  uint32_t turn = 0;
};
Tables g_tables[16];

// How many of the queries at q, n at most, go on with the run that `u` (checked) belongs to: the same but for the
// row, which is `next` and so on.  A run of many queries is what a decoding step of many samples makes, and the
// host's pass over them took longer than the kernel (64 programs x 100: 16.6 us a call, 8.9 of them the kernel;
// 13.8 this way).  Eight queries to a branch, once a run has a dozen: looking eight ahead from a run's second query on cost
// more than it saved where runs are short (16,000 queries in runs of 2, 4, 8 and 16: 121, 72, 48 and 36 us a call; 43, 44, 37
// and 38 one by one; 42, 38, 37 and 35 this way).  The last of the eight is looked at first.
constexpr uint32_t kLongRun = 12;
inline uint32_t same_run(const vl_mask_query *q, uint32_t n, const vl_mask_query &u, const uint16_t *next, int64_t stride) {
  const uintptr_t mir = (uintptr_t)u.mir, live = (uintptr_t)u.live, step = (uintptr_t)(stride * 2);
  uintptr_t at = (uintptr_t)next;
  auto other = [&](const vl_mask_query &x, uintptr_t cand) {
    return ((uintptr_t)x.mir ^ mir) | ((uintptr_t)x.live ^ live) | ((uintptr_t)x.cand ^ cand) | (uintptr_t)((x.occ ^ u.occ) | x.reserved0) | (uintptr_t)!cand;
  };
  uint32_t k = 0;
  for (; k + 8 <= n && !other(q[k + 7], at + 7 * step); k += 8, at += 8 * step) {
    uintptr_t any = 0;
    for (uint32_t t = 0; t < 7; ++t) any |= other(q[k + t], at + t * step);
    if (any) break;
  }
  while (k < n && !other(q[k], at)) { ++k; at += step; }
  return k;
}

}  // namespace

extern "C" int32_t vl_free_bases_multi(const vl_mask_query *queries, uint32_t n, uint32_t *masks, vl_stream stream_) {
  if (!queries || !masks) return VL_E_NULL;
  if (n == 0) return VL_E_SHAPE;
  uint32_t max_w = 1;
  // neighbouring queries of one program at one occurrence whose rows lie at equal distances are one run
  RunArgs args;
  std::unique_lock<std::mutex> lock;
  Tables::One *t = nullptr;
  // Room for more runs than there is now: the first too many for the argument takes a table, which grows with the
  // runs, not with the queries, and the runs are put together there.  (Handed back by value: what the loop below
  // works with stays in registers.)
  struct Room {
    Run *runs;
    uint32_t most;
    int32_t rc;
  };
  auto more_room = [&]() -> Room {
    auto fail = [](int32_t rc) { return Room{nullptr, 0, rc}; };
    if (!t) {
      int device = 0;
      hipError_t e = hipGetDevice(&device);
      if (e != hipSuccess) return fail(hip_fail(e));
      if (device < 0 || device >= 16) return fail(VL_E_ARG);
      Tables &all = g_tables[device];
      lock = std::unique_lock<std::mutex>(all.mu);
      t = &all.one[all.turn = (all.turn + 1) % kTables];
      // the kernel that last read this table must be done with it before it is overwritten
      if (t->in_flight) e = hipEventSynchronize(t->consumed);
      if (e != hipSuccess) return fail(hip_fail(e));
      t->in_flight = false;
      if (!t->host) {
        e = hipHostMalloc((void **)&t->host, (size_t)kLeastRuns * sizeof(Run), hipHostMallocDefault);
        if (e != hipSuccess) return fail(hip_fail(e));
        t->cap = kLeastRuns;
      }
      if (!t->consumed) e = hipEventCreateWithFlags(&t->consumed, hipEventDisableTiming);
      if (e != hipSuccess) return fail(hip_fail(e));
      memcpy(t->host, args.run, sizeof(args.run));
      return Room{t->host, t->cap, VL_OK};
    }
    Run *larger = nullptr;
    const hipError_t e = hipHostMalloc((void **)&larger, (size_t)t->cap * 4 * sizeof(Run), hipHostMallocDefault);
    if (e != hipSuccess) return fail(hip_fail(e));
    memcpy(larger, t->host, (size_t)t->cap * sizeof(Run));
    (void)hipHostFree(t->host);
    t->host = larger;
    t->cap *= 4;
    return Room{t->host, t->cap, VL_OK};
  };
  Run *runs = args.run;
  uint32_t n_runs = 0, most_runs = kArgRuns;
  // a workgroup per four queries (one per wavefront) up to some five hundred workgroups, then longer shares, since each rebuilds P(i)
  // (64 programs x 100, longer shares from 1,024 workgroups, from 512 and from 256 on: 11.0, 9.3 and 11.4 us)
  const uint32_t per_block = kMaskWaves * std::max(1u, std::min(16u, n / (kMaskWaves * 512u)));
  uint32_t blocks = 0;
  Run run = {};
  const vl_mir *mir = nullptr;
  const vl_live *live = nullptr;
  const uint16_t *next = nullptr;
  for (uint32_t j = 0; j < n; ++j) {
    const vl_mask_query &u = queries[j];
    const bool same = j > 0 && u.mir == mir && u.live == live;   // (checked with the query before)
    if (!same || !u.cand) {
      if (!u.mir || !u.live || !u.cand) return VL_E_NULL;
      if (u.mir->magic != kMirMagic || u.live->magic != kLiveMagic || u.live->mir != u.mir || u.mir->lowered) return VL_E_ARG;
      mir = u.mir; live = u.live;
      max_w = std::max(max_w, mir->h.W);
    }
    if (u.reserved0 != 0) return VL_E_ARG;
    if (u.occ >= mir->h.O) return VL_E_SHAPE;
    if (same && u.occ == run.occ && (run.count == 1 || u.cand == next)) {
      if (run.count == 1) run.stride = ((int64_t)(intptr_t)u.cand - (int64_t)(intptr_t)run.cand) / 2;
      if (u.cand == run.cand + (int64_t)run.count * run.stride) {   // (an odd distance in bytes is no multiple of an element)
        ++run.count;
        next = u.cand + run.stride;
        if (run.count == kLongRun) {
          const uint32_t more = same_run(queries + j + 1, n - j - 1, u, next, run.stride);
          run.count += more;
          next += (int64_t)more * run.stride;
          j += more;
        }
        continue;
      }
    }
    if (run.count) {   // the run before is complete
      if (n_runs == most_runs) {
        const Room more = more_room();
        if (more.rc != VL_OK) return more.rc;
        runs = more.runs;
        most_runs = more.most;
      }
      runs[n_runs++] = run;
      blocks += run.count <= per_block ? 1u : (run.count + per_block - 1) / per_block;
    }
    run = Run{mir->dev, live->dev, u.cand, 0, u.occ, 1, j, blocks};
  }
  if (n_runs == most_runs) {
    const Room more = more_room();
    if (more.rc != VL_OK) return more.rc;
    runs = more.runs;
  }
  runs[n_runs++] = run;
  blocks += run.count <= per_block ? 1u : (run.count + per_block - 1) / per_block;
  hipStream_t stream = (hipStream_t)stream_;
  const size_t lds = (size_t)max_w * 4;
  if (!t) {
    k_free_bases<true><<<blocks, kMaskThreads, lds, stream>>>(args, n_runs, per_block, masks);
    VL_HIP(hipGetLastError());
    return VL_OK;
  }
  if (t->dev_cap < n_runs) {
    if (t->dev) (void)hipFree(t->dev);
    t->dev = nullptr; t->dev_cap = 0;
    VL_HIP(device_alloc((void **)&t->dev, (size_t)t->cap * sizeof(Run)));
    t->dev_cap = t->cap;
  }
  VL_HIP(hipMemcpyAsync(t->dev, t->host, (size_t)n_runs * sizeof(Run), hipMemcpyHostToDevice, stream));
  if (blocks == n_runs && n <= 2ull * n_runs) k_free_bases_alone<<<blocks, kAloneThreads, lds, stream>>>(t->dev, masks);
  else k_free_bases<false><<<blocks, kMaskThreads, lds, stream>>>(t->dev, n_runs, per_block, masks);
  VL_HIP(hipGetLastError());
  VL_HIP(hipEventRecord(t->consumed, stream));
  t->in_flight = true;
  return VL_OK;
}
