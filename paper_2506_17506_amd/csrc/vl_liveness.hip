// Liveness analysis on the GPU, batched over kernels (one grid slice per kernel).
//
// Pipeline (every step is a kernel below; the host only sizes buffers):
//   1. group operand occurrences by vreg (large programs: count / scan / place / sort)
//   2. put them in order; per-block use and def bitsets from the first mention of each vreg in a block
//   3. backward dataflow to the least fixed point, one bitset word per lane
//   4. per occurrence: liveness after its instruction, kill flag, and its role in
//      the verifier's event stream
//   5. count, prefix and write the event stream, the live intervals and the
//      per-tile live-in lists; optionally the dense per-point bitsets
// The paper defers this to "following the control and data dependency"
// (Section 4.6); the dataflow equations are the textbook ones its Safety
// condition (Section 3.4) needs to know which lifetimes overlap.
#include <algorithm>
#include <cstring>
#include <initializer_list>
#include <mutex>
#include <new>
#include <vector>

#include "vl_dev.h"

using namespace vl;

// The tables of a launch's programs hold the structures themselves: nothing but the kernel's arguments is
// read before an array's address is known, and the loads are scalar ones wherever they stand.  (A launch
// of few programs is a chain of some six trips to memory of 0.8 us, its table of pointers was one.)
#define MIRS const DevProg *__restrict__ mirs, const DevLive *__restrict__ lives

namespace {

// Which program and which of its blocks a workgroup of a two-dimensional launch has.  Consecutive
// workgroups go to the eight dies in turn, each with an L2 of its own; where a batch deals its programs out
// to the dies (`deal`), program p stays on die p % 8 through the launches from k_order on and k_group (not the scans, nor
// those that only very large programs have), so that what its workgroups
// gather and scatter meets in one L2: row y of the grid then holds programs 8 y to 8 y + 7 side by side.
// (256 programs of 1,000-20,000 instructions, us per launch, spread over all dies and dealt out: k_group 50 and 31,
// k_events 98 and 78, k_stage_count 35 and 29, k_stage_finish 30 and 21.)
struct Grid { uint32_t n, dealt; };   // programs; 3 where they are dealt out, else 0
__device__ inline uint32_t grid_prog(Grid g) { return g.dealt ? blockIdx.y * 8u + (blockIdx.x & 7u) : blockIdx.y; }
__device__ inline uint32_t grid_block(Grid g) { return blockIdx.x >> g.dealt; }

template <class P> __device__ inline bool bit_get(P row, uint32_t v) { return (row[v >> 5] >> (v & 31)) & 1u; }

// first of the entries [lo, hi) of a vreg that is at instruction `at` or later
__device__ inline uint32_t first_entry_at(const DevLive VL_CONSTANT &L, uint32_t lo, uint32_t hi, uint32_t at) {
  while (lo < hi) {
    uint32_t mid = (lo + hi) >> 1;
    if ((L.ent[mid].y >> 2) < at) lo = mid + 1; else hi = mid;
  }
  return lo;
}

// ---- 1. occurrences grouped by vreg -------------------------------------------------
constexpr uint32_t kSlice = 8192;   // occurrences per workgroup in the counting kernels

// A slice's counts where a word for every vreg would not fit LDS: a table with a place per vreg modulo its size, which
// belongs to the first vreg of the slice that asks for it.  Others that fall on the place go to memory one by one, but the vregs
// that are mentioned again and again nearly always get a place.  (What bounds these launches is atomics on those few counters,
// of all workgroups at a time: with every occurrence counted and placed in memory, 8 programs of 112,000 instructions took 783 us an
// analysis, and 824 once workgroups had their addresses without a trip to memory and met at the counters sooner; 318 this way.
// One program of 50,000: 353 and 188.  Where no vreg is mentioned more than others, it costs what it saves: 8 programs of
// 200,000 occurrences, both launches 139 and 140.)
constexpr uint32_t kPlaces = 8192;
struct CountTable {
  uint32_t *const vreg, *const count;
  __device__ explicit CountTable(uint32_t *lds) : vreg(lds), count(lds + kPlaces) {}
  __device__ void clear(uint32_t tid) {
    for (uint32_t x = tid; x < kPlaces; x += 1024) { vreg[x] = kNone; count[x] = 0; }
  }
  __device__ bool claim(uint32_t v) {
    const uint32_t owner = atomicCAS(&vreg[v % kPlaces], kNone, v);
    return owner == kNone || owner == v;
  }
  __device__ bool has(uint32_t v) const { return vreg[v % kPlaces] == v; }
  __device__ uint32_t &of(uint32_t v) { return count[v % kPlaces]; }
};

// Occurrences per vreg.  A few vregs (base addresses, accumulators) are mentioned
// thousands of times, so each workgroup first counts its slice in LDS, in a histogram over all vregs or in a
// CountTable, and then adds the non-zero bins to the global counters once.
template <bool kLds>
__global__ __launch_bounds__(1024) void k_count(MIRS) {
  const DevProg VL_CONSTANT &m = as_constant(mirs)[blockIdx.y];
  const DevLive VL_CONSTANT &L = as_constant(lives)[blockIdx.y];
  extern __shared__ uint32_t sm[];
  const uint32_t o0 = blockIdx.x * kSlice;
  if (o0 >= m.O) return;
  const uint32_t o1 = min(m.O, o0 + kSlice);
  if (!kLds) {
    CountTable table(sm);
    table.clear(threadIdx.x);
    __syncthreads();
    for (uint32_t o = o0 + threadIdx.x; o < o1; o += 1024) {
      const uint32_t v = m.occ_vreg[o];
      if (table.claim(v)) atomicAdd(&table.of(v), 1u);
      else atomicAdd(&L.vcnt[v], 1u);
    }
    __syncthreads();
    for (uint32_t x = threadIdx.x; x < kPlaces; x += 1024)
      if (table.count[x]) atomicAdd(&L.vcnt[table.vreg[x]], table.count[x]);
    return;
  }
  for (uint32_t v = threadIdx.x; v < m.V; v += 1024) sm[v] = 0;
  __syncthreads();
  for (uint32_t o = o0 + threadIdx.x; o < o1; o += 1024) atomicAdd(&sm[m.occ_vreg[o]], 1u);
  __syncthreads();
  for (uint32_t v = threadIdx.x; v < m.V; v += 1024)
    if (sm[v]) atomicAdd(&L.vcnt[v], sm[v]);
}

constexpr uint32_t kShortList = 16;   // longer occurrence lists go to the bitmap sort

// inclusive prefix over the wavefront, in the vector unit (rows of 16 lanes, then across rows)
__device__ inline uint32_t wave_prefix(uint32_t x) {
  x += __builtin_amdgcn_update_dpp(0u, x, 0x111, 0xf, 0xf, false);   // row_shr:1, 2, 4, 8
  x += __builtin_amdgcn_update_dpp(0u, x, 0x112, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0u, x, 0x114, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0u, x, 0x118, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0u, x, 0x142, 0xa, 0xf, false);   // row_bcast:15 into rows 1 and 3
  x += __builtin_amdgcn_update_dpp(0u, x, 0x143, 0xc, 0xf, false);   // row_bcast:31 into rows 2 and 3
  return x;
}

constexpr uint32_t kStretch = 256;    // entries or instructions whose counts are prefixed by the kernel that counts them
__host__ __device__ inline uint32_t stretches(uint32_t n) { return (n + kStretch - 1) / kStretch; }

enum { kScanVreg = 0, kScanItems = 1, kScanSeg = 2, kScanSeed = 3, kScanBound = 4 };   // kScanItems, kScanSeg: totals of stretches

// In-place exclusive scan of p[0..n), total to p[n]; one 1024-thread block per kernel.
// (The array is chosen at compile time: a run-time switch over the four arrays was
// seen to pick the wrong pointer in its default branch.)
template <int kWhich>
__device__ inline void f_scan(const DevProg VL_CONSTANT &m, const DevLive VL_CONSTANT &L) {
  uint32_t VL_GLOBAL *p = kWhich == kScanVreg ? L.vcnt : kWhich == kScanItems ? L.item_base : kWhich == kScanSeg ? L.seg_base :
                          kWhich == kScanBound ? L.bound_off : L.seed_off;
  const uint32_t n = kWhich == kScanVreg ? m.V : kWhich == kScanItems ? stretches(m.N) : kWhich == kScanSeg ? stretches(m.O) :
                     kWhich == kScanBound ? m.B : L.T;
  // Each of the 16 wavefronts owns a contiguous sixteenth of the array and walks it 256
  // elements at a time (four consecutive elements per lane, one 16-byte access): first to
  // total its part, then, once the parts' totals are prefixed, to write the exclusive sums.
  __shared__ uint32_t part[16];
  const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
  const uint32_t per = ((n + 15u) / 16u + 255u) & ~255u;
  const uint32_t lo = min(n, wave * per), hi = min(n, lo + per);
  auto load4 = [&](uint32_t i) {
    u32x4 x = 0;
    if (i + 4 <= hi) x = *reinterpret_cast<const u32x4 VL_GLOBAL *>(p + i);
    else {
      if (i < hi) x.x = p[i];
      if (i + 1 < hi) x.y = p[i + 1];
      if (i + 2 < hi) x.z = p[i + 2];
    }
    return x;
  };
  uint32_t sum = 0;
  for (uint32_t i = lo + lane * 4; i < hi; i += 4 * 256) {   // four reads in flight
    u32x4 x[4];
#pragma unroll
    for (uint32_t u = 0; u < 4; ++u) x[u] = load4(i + u * 256);   // zeros beyond hi
#pragma unroll
    for (uint32_t u = 0; u < 4; ++u) sum += x[u].x + x[u].y + x[u].z + x[u].w;
  }
  for (int d = 32; d >= 1; d >>= 1) sum += (uint32_t)__shfl_xor((int)sum, d, 64);
  if (lane == 0) part[wave] = sum;
  __syncthreads();
  uint32_t base = 0, total = 0;
  for (uint32_t k = 0; k < 16; ++k) {
    if (k < wave) base += part[k];
    total += part[k];
  }
  for (uint32_t i00 = lo; i00 < hi; i00 += 4 * 256) {
    u32x4 ahead[4];   // the array is rewritten in place: the reads of four rounds go before their writes
#pragma unroll
    for (uint32_t u = 0; u < 4; ++u) ahead[u] = load4(i00 + u * 256 + lane * 4);
#pragma unroll
    for (uint32_t u = 0; u < 4; ++u) {
      const uint32_t i0 = i00 + u * 256;
      if (i0 >= hi) break;
      const uint32_t i = i0 + lane * 4;
      const u32x4 x = ahead[u];
      const uint32_t s4 = x.x + x.y + x.z + x.w;
      uint32_t incl = s4;
      for (int d = 1; d < 64; d <<= 1) {
        const uint32_t y = (uint32_t)__shfl_up((int)incl, d, 64);
        if ((int)lane >= d) incl += y;
      }
      const uint32_t e0 = base + incl - s4;
      const u32x4 out = {e0, e0 + x.x, e0 + x.x + x.y, e0 + x.x + x.y + x.z};
      if (kWhich == kScanVreg) {   // the counts are list lengths: queue the lists the bitmap sort will take
        if (x.x > kShortList) L.long_queue[atomicAdd(&L.counters[kCtrLong], 1u)] = i;
        if (x.y > kShortList) L.long_queue[atomicAdd(&L.counters[kCtrLong], 1u)] = i + 1;
        if (x.z > kShortList) L.long_queue[atomicAdd(&L.counters[kCtrLong], 1u)] = i + 2;
        if (x.w > kShortList) L.long_queue[atomicAdd(&L.counters[kCtrLong], 1u)] = i + 3;
      }
      if (i + 4 <= hi) *reinterpret_cast<u32x4 VL_GLOBAL *>(p + i) = out;
      else {
        if (i < hi) p[i] = out.x;
        if (i + 1 < hi) p[i + 1] = out.y;
        if (i + 2 < hi) p[i + 2] = out.z;
      }
      base += (uint32_t)__shfl((int)incl, 63, 64);
    }
  }
  if (threadIdx.x == 0) p[n] = total;
}

template <int kWhich>
__global__ __launch_bounds__(1024) void k_scan(MIRS) {
  f_scan<kWhich>(as_constant(mirs)[blockIdx.x], as_constant(lives)[blockIdx.x]);
}

// Places each occurrence into its vreg's range (order inside a range is fixed later).
// Same privatisation: the slice reserves a sub-range per vreg with one global atomic,
// then ranks its own occurrences in LDS; those without a place in the table reserve one by one.
template <bool kLds>
__global__ __launch_bounds__(1024) void k_place(MIRS) {
  const DevProg VL_CONSTANT &m = as_constant(mirs)[blockIdx.y];
  const DevLive VL_CONSTANT &L = as_constant(lives)[blockIdx.y];
  extern __shared__ uint32_t sm[];
  const uint32_t o0 = blockIdx.x * kSlice;
  if (o0 >= m.O) return;
  const uint32_t o1 = min(m.O, o0 + kSlice);
  if (!kLds) {
    CountTable table(sm);
    table.clear(threadIdx.x);
    __syncthreads();
    for (uint32_t o = o0 + threadIdx.x; o < o1; o += 1024) {
      const uint32_t v = m.occ_vreg[o];
      if (table.claim(v)) atomicAdd(&table.of(v), 1u);
    }
    __syncthreads();
    for (uint32_t x = threadIdx.x; x < kPlaces; x += 1024) {
      const uint32_t c = table.count[x], v = table.vreg[x];
      if (c) table.count[x] = L.vcnt[v] + atomicAdd(&L.vcur[v], c);
    }
    __syncthreads();
    for (uint32_t o = o0 + threadIdx.x; o < o1; o += 1024) {
      const uint32_t v = m.occ_vreg[o];
      L.vocc_tmp[table.has(v) ? atomicAdd(&table.of(v), 1u) : L.vcnt[v] + atomicAdd(&L.vcur[v], 1u)] = o;
    }
    return;
  }
  // one word per vreg: first the slice's count, then the next free position of the
  // sub-range reserved for the slice
  uint32_t *cnt = sm;
  for (uint32_t v = threadIdx.x; v < m.V; v += 1024) cnt[v] = 0;
  __syncthreads();
  for (uint32_t o = o0 + threadIdx.x; o < o1; o += 1024) atomicAdd(&cnt[m.occ_vreg[o]], 1u);
  __syncthreads();
  for (uint32_t v = threadIdx.x; v < m.V; v += 1024) {
    const uint32_t c = cnt[v];
    if (c) cnt[v] = L.vcnt[v] + atomicAdd(&L.vcur[v], c);
  }
  __syncthreads();
  for (uint32_t o = o0 + threadIdx.x; o < o1; o += 1024) L.vocc_tmp[atomicAdd(&cnt[m.occ_vreg[o]], 1u)] = o;
}

// Lists of up to kShortList occurrences are rank-sorted by one lane (the longer ones were
// queued by the scan of the list lengths).
__device__ inline void f_sort_short(const DevProg VL_CONSTANT &m, const DevLive VL_CONSTANT &L, const uint32_t bx, const uint32_t tx) {
  const uint32_t v = bx * 256 + tx;
  if (v >= m.V) return;
  const uint32_t lo = L.vcnt[v], len = L.vcnt[v + 1] - lo;
  if (len == 0) { L.first[v] = kNone; return; }
  if (len > kShortList) return;
  auto put = [&](uint32_t at, uint32_t x) { L.vocc[at] = x; };
  if (len <= 8) {
    // the common case: all loads issued at once, ranks computed in registers (absent
    // elements are larger than any occurrence index)
    uint32_t a[8];
#pragma unroll
    for (uint32_t k = 0; k < 8; ++k) a[k] = k < len ? L.vocc_tmp[lo + k] : kNone;
#pragma unroll
    for (uint32_t j = 0; j < 8; ++j) {
      uint32_t r = 0;
#pragma unroll
      for (uint32_t k = 0; k < 8; ++k) r += a[k] < a[j];
      if (j < len) put(lo + r, a[j]);
    }
    return;
  }
  // up to kShortList: the same with twice the registers (a lane or two of most wavefronts)
  static_assert(kShortList <= 16, "the register sort holds 16 occurrences");
  uint32_t a[16];
#pragma unroll
  for (uint32_t k = 0; k < 16; ++k) a[k] = k < len ? L.vocc_tmp[lo + k] : kNone;
#pragma unroll
  for (uint32_t j = 0; j < 16; ++j) {
    uint32_t r = 0;
#pragma unroll
    for (uint32_t k = 0; k < 16; ++k) r += a[k] < a[j];
    if (j < len) put(lo + r, a[j]);
  }
}

constexpr uint32_t kBitmapWords = 2048;              // 8 KB of LDS
constexpr uint32_t kBitmapSpan = kBitmapWords * 32;  // occurrences per window
constexpr uint32_t kLongBlocks = 64;                 // workgroups per kernel that take long lists

// Long lists: occurrence indices are distinct, so marking them in a bitmap and reading
// the bitmap back in order sorts them, one window of kBitmapSpan occurrences at a time.
__device__ inline void f_sort_long(const DevProg VL_CONSTANT &m, const DevLive VL_CONSTANT &L, const uint32_t bx, const uint32_t tid) {
  __shared__ uint32_t bm[kBitmapWords];
  __shared__ uint32_t wave_total[4];
  const uint32_t n_long = L.counters[kCtrLong];
  const uint32_t lane = tid & 63u, wave = tid >> 6;
  for (uint32_t q = bx; q < n_long; q += kLongBlocks) {
    const uint32_t v = L.long_queue[q];
    const uint32_t lo = L.vcnt[v], len = L.vcnt[v + 1] - lo;
    uint32_t written = 0;
    for (uint32_t wb = 0; wb < m.O; wb += kBitmapSpan) {
      const uint32_t span = min(kBitmapSpan, m.O - wb), nw = (span + 31u) / 32u;
      for (uint32_t w = tid; w < nw; w += 256) bm[w] = 0;
      __syncthreads();
      for (uint32_t j = tid; j < len; j += 256) {
        uint32_t x = L.vocc_tmp[lo + j] - wb;
        if (x < span) atomicOr(&bm[x >> 5], 1u << (x & 31));
      }
      __syncthreads();
      const uint32_t chunk = (nw + 255u) / 256u;
      const uint32_t w0 = min(nw, tid * chunk), w1 = min(nw, w0 + chunk);
      uint32_t cnt = 0;
      for (uint32_t w = w0; w < w1; ++w) cnt += __popc(bm[w]);
      // exclusive prefix of cnt over the 256 threads: within the wavefront by shuffles,
      // across the four wavefronts through LDS
      uint32_t incl = cnt;
      for (int d = 1; d < 64; d <<= 1) {
        const uint32_t y = (uint32_t)__shfl_up((int)incl, d, 64);
        if ((int)lane >= d) incl += y;
      }
      if (lane == 63) wave_total[wave] = incl;
      __syncthreads();
      uint32_t before = 0, total = 0;
      for (uint32_t k = 0; k < 4; ++k) {
        if (k < wave) before += wave_total[k];
        total += wave_total[k];
      }
      uint32_t pos = lo + written + before + incl - cnt;
      for (uint32_t w = w0; w < w1; ++w) {
        uint32_t bits = bm[w];
        while (bits) {
          uint32_t b = __ffs(bits) - 1;
          bits &= bits - 1;
          uint32_t x = wb + w * 32 + b;
          L.vocc[pos++] = x;
        }
      }
      written += total;
      __syncthreads();
    }
  }
}

// both sorts in one launch: the first kLongBlocks workgroups of each kernel take the long lists
__global__ __launch_bounds__(256) void k_sort(MIRS) {
  const DevProg VL_CONSTANT &m = as_constant(mirs)[blockIdx.y];
  const DevLive VL_CONSTANT &L = as_constant(lives)[blockIdx.y];
  if (blockIdx.x < kLongBlocks) f_sort_long(m, L, blockIdx.x, threadIdx.x);
  else f_sort_short(m, L, blockIdx.x - kLongBlocks, threadIdx.x);
}

// The usual way: a workgroup per `slice` occurrences of a program (2,048 to 16,384), all of which count the whole
// program: the LDS of each then holds, a word per vreg, first the list lengths, then the lists'
// starts, then the places its own occurrences go to (the starts plus what earlier workgroups place;
// kPacked: up to 65,535 occurrences, whose count and whose count in earlier slices share a word, otherwise those are counted anew),
// and nothing is cleared, reserved or prefixed in memory, nor in a launch of its own.  Occurrences
// are placed 1,024 at a time, with a barrier in between: what is out of order in a list
// afterwards lies within one such round, and the next kernel puts it right.  It also clears what
// the later kernels add to.
// What bounds it: LDS atomics and the placing stores, 64 lines per wavefront, of the largest
// programs (256 programs of 1,000-20,000 instructions: 31 us, 50 before programs were dealt out to the dies; a
// workgroup per program 58 us then; clearing, counting, scanning and placing in launches of their own 86 us).
constexpr uint32_t kRound = 1024;
constexpr uint32_t kGroupRounds = 16;         // most rounds of a workgroup, one after the other
// Few programs are cut into more slices, of fewer rounds, while there are compute units for them; up to eight of a
// program, since each reads and counts the whole of it.
constexpr uint32_t kGroupFew = 256, kGroupSlices = 8;
constexpr uint32_t kGroupMaxOcc = 1u << 17;   // with more in some program, counting it all in every workgroup costs too much
template <bool kPacked>
__global__ __launch_bounds__(1024) void k_group(MIRS, const Grid grid, const uint32_t slice) {
  const uint32_t prog = grid_prog(grid), bx = grid_block(grid);
  if (prog >= grid.n) return;
  const DevProg VL_CONSTANT &m = as_constant(mirs)[prog];
  const DevLive VL_CONSTANT &L = as_constant(lives)[prog];
  extern __shared__ uint32_t sm[];   // [V]
  __shared__ uint32_t part[16];
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
  const uint32_t s0 = bx * slice, n_slices = max(1u, (m.O + slice - 1) / slice), s1 = min(m.O, s0 + slice);
  if (bx >= n_slices) return;
  auto add_all = [&](uint32_t end) {   // sm[v] += mentions among the occurrences [0, end); kPacked: high half, those before the slice
    for (uint32_t o = tid * 4; o < end; o += 4 * 4 * 1024) {
      u32x4 v[4];
#pragma unroll
      for (uint32_t u = 0; u < 4; ++u) {
        const uint32_t x = o + u * 4 * 1024;
        v[u] = kNone;
        if (x + 4 <= end) v[u] = *reinterpret_cast<const u32x4 VL_GLOBAL *>(m.occ_vreg + x);
        else {
          if (x < end) v[u].x = m.occ_vreg[x];
          if (x + 1 < end) v[u].y = m.occ_vreg[x + 1];
          if (x + 2 < end) v[u].z = m.occ_vreg[x + 2];
        }
      }
#pragma unroll
      for (uint32_t u = 0; u < 4; ++u)
#pragma unroll
        for (uint32_t t = 0; t < 4; ++t)   // (a slice begins at a multiple of four)
          if (v[u][t] != kNone) atomicAdd(&sm[v[u][t]], kPacked && o + u * 4 * 1024 < s0 ? 0x10001u : 1u);
    }
  };
  for (uint32_t v = tid; v < m.V; v += 1024) sm[v] = 0;
  __syncthreads();
  add_all(m.O);
  // (the regions are whole vectors long)
  const uint32_t vecs = (m.B * m.W + 3u) / 4u;
  const u32x4 none = {0, 0, 0, 0};
  for (uint32_t x = bx * 1024 + tid; x < vecs; x += n_slices * 1024) {
    reinterpret_cast<u32x4 VL_GLOBAL *>(L.use)[x] = none;
    reinterpret_cast<u32x4 VL_GLOBAL *>(L.def)[x] = none;
    reinterpret_cast<u32x4 VL_GLOBAL *>(L.live_in)[x] = none;
  }
  if (bx == 0 && tid < kCounters) L.counters[tid] = 0;
  __syncthreads();
  // exclusive prefix: a contiguous run of vregs per thread
  const uint32_t per = (m.V + 1023u) / 1024u, lo = min(m.V, tid * per), hi = min(m.V, lo + per);
  uint32_t sum = 0;
#pragma unroll 4
  for (uint32_t v = lo; v < hi; ++v) sum += kPacked ? sm[v] & 0xFFFFu : sm[v];
  uint32_t incl = sum;
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t y = (uint32_t)__shfl_up((int)incl, d, 64);
    if ((int)lane >= d) incl += y;
  }
  if (lane == 63) part[wave] = incl;
  __syncthreads();
  uint32_t run = incl - sum;
  for (uint32_t k = 0; k < wave; ++k) run += part[k];
#pragma unroll 4
  for (uint32_t v = lo; v < hi; ++v) {
    const uint32_t c = sm[v];
    sm[v] = kPacked ? run | (c & 0xFFFF0000u) : run;
    run += kPacked ? c & 0xFFFFu : c;
  }
  __syncthreads();
  for (uint32_t v = bx * 1024 + tid; v < m.V; v += n_slices * 1024) {
    const uint32_t start = sm[v], after = v + 1 < m.V ? sm[v + 1] : m.O;
    const uint32_t at = kPacked ? start & 0xFFFFu : start, next = kPacked ? after & 0xFFFFu : after;
    L.vcnt[v] = at;
    L.last_live[v] = 0;
    if (at == next) L.first[v] = kNone;
  }
  if (bx == 0 && tid == 0) L.vcnt[m.V] = m.O;
  __syncthreads();
  if (kPacked) {
    for (uint32_t v = tid; v < m.V; v += 1024) sm[v] = (sm[v] & 0xFFFFu) + (sm[v] >> 16);
  } else {
    add_all(min(s0, m.O));
  }
  __syncthreads();
  // the vregs of the next two rounds are in flight
  auto vreg_of = [&](uint32_t o) { return o < s1 ? m.occ_vreg[o] : 0u; };
  uint32_t v0 = vreg_of(s0 + tid), v1 = vreg_of(s0 + kRound + tid);
  for (uint32_t o0 = s0; o0 < s1; o0 += kRound) {
    const uint32_t v2 = vreg_of(o0 + 2 * kRound + tid), o = o0 + tid;
    if (o < s1) L.vocc_tmp[atomicAdd(&sm[v0], 1u)] = o;
    v0 = v1;
    v1 = v2;
    // the round's places are taken before the next round takes any (no wait for the stores)
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  }
}

// ---- 2. entries in order, block summaries -------------------------------------------------
// A workgroup takes a stretch of the grouped occurrences, puts it in order, writes the entry records
// and collects its share of the block summaries.
//
// Order: a list is a row of groups, one per round of 1,024 occurrences in which it was filled;
// groups follow each other, inside a group the order is open.  An entry's place is its group's
// first plus the smaller ones in the group (some six entries, read from LDS, where the stretch
// lies with a margin on both sides; where groups begin is a bit per place).  A group that reaches beyond the margin (a value mentioned more than a hundred times in
// 1,024 occurrences) is ranked by a bitmap of its round.  kSorted: the lists already ascend (the
// large-program sort ran).
//
// Summaries: def[b]: vregs written in b.  use[b]: vregs whose first mention in b reads them
// (an instruction reads before it writes).  The stretch's vregs span a narrow range of bitset
// words; the bits are collected in an LDS table [block][word of the range] and each non-zero word
// goes to memory once; when the table would not fit, every entry issues its own atomics.
//
// (A launch that sorted each list in the registers of a lane and one that summarised the sorted
// entries took 38 and 45 us, this 70 then and 59 now, but this needs no sorted list and no cleared counters.)
constexpr uint32_t kOrdStretch = 1024;
constexpr uint32_t kOrdBack = 72;        // entries before the stretch that are put in order too: one more than an instruction has
constexpr uint32_t kOrdMargin = 128;
constexpr uint32_t kOrdWindow = kOrdBack + kOrdStretch + 2 * kOrdMargin;
constexpr uint32_t kOrdWords = kOrdStretch / 32 + 1;   // most words a stretch touches when every vreg is mentioned
static_assert(kOrdBack > kMaxOperands, "the look-back has to leave an instruction");

// Threads of a workgroup: 512 (the sweep of 256 programs: 60 us a launch; 66 with 256, 81 with 1,024, of which
// a compute unit holds two workgroups); 1,024 where the launch has no more workgroups than the device
// holds at once and a workgroup's chain is what it takes (8,000 instructions: 8.2 us, 9.7 with 512, 14.2 with
// 256; 2,000: 6.6, 8.4, 11.9).
constexpr uint32_t kOrdFew = 512;   // workgroups of 1,024 threads that the device holds
template <bool kSorted, uint32_t kOrdThreads>
__global__ __launch_bounds__(kOrdThreads) void k_order(MIRS, const Grid grid, const uint32_t lds_words) {
  const uint32_t prog = grid_prog(grid), bx = grid_block(grid);
  if (prog >= grid.n) return;
  const DevProg VL_CONSTANT &m = as_constant(mirs)[prog];
  const DevLive VL_CONSTANT &L = as_constant(lives)[prog];
  extern __shared__ uint32_t sm[];
  constexpr uint32_t kOrdPer = (kOrdWindow + kOrdThreads - 1) / kOrdThreads;
  // by place in the window; s_o holds the occurrences as they stand, then in order with kRecKeeps
  __shared__ uint32_t s_o[kOrdWindow], s_v[kOrdWindow], s_ifl[kOrdWindow], s_blk[kOrdWindow];
  __shared__ uint32_t heads[kOrdPer * kOrdThreads / 32 + 1];   // a bit per place: a group begins here
  __shared__ uint32_t bits[kRound / 32], n_edge, crossing;
  const uint32_t s0 = bx * kOrdStretch, tid = threadIdx.x;
  if (s0 >= m.O) return;
  const uint32_t s1 = min(m.O, s0 + kOrdStretch);
  const uint32_t x_lo = s0 - min(s0, kOrdBack);                                           // first entry put in order
  const uint32_t w_lo = x_lo - min(x_lo, kOrdMargin), w_hi = min(m.O, s1 + kOrdMargin);   // the window
  const uint32_t n_win = w_hi - w_lo;
  const uint32_t VL_GLOBAL *const src = kSorted ? L.vocc : L.vocc_tmp;
  uint32_t o[kOrdPer], v[kOrdPer], ifl[kOrdPer], to[kOrdPer];   // v with kRecKeeps
  {
    uint64_t rec[kOrdPer];
#pragma unroll
    for (uint32_t u = 0; u < kOrdPer; ++u) {
      const uint32_t r = u * kOrdThreads + tid;
      o[u] = r < n_win ? src[w_lo + r] : kNone;
    }
#pragma unroll
    for (uint32_t u = 0; u < kOrdPer; ++u) rec[u] = o[u] != kNone ? m.occ_rec[o[u]] : 0ull;
#pragma unroll
    for (uint32_t u = 0; u < kOrdPer; ++u) {
      const uint32_t r = u * kOrdThreads + tid;
      v[u] = (uint32_t)rec[u];
      ifl[u] = (uint32_t)(rec[u] >> 32);
      if (r < n_win) { s_o[r] = o[u]; s_v[r] = v[u] & ~kRecKeeps; }
    }
  }
  if (tid == 0) { crossing = 0; n_edge = 0; }
  if (tid < kRound / 32) bits[tid] = 0;
  __syncthreads();
  // the range of bitset words is known once the vregs are staged (putting a list in order leaves each
  // place its vreg): the table is cleared exactly as far as it will be used.  Vregs that are never mentioned
  // take no entries but widen the range, and the launch's LDS is sized by its largest program
  const uint32_t word0 = s_v[s0 - w_lo] >> 5, n_words = (s_v[s1 - 1 - w_lo] >> 5) - word0 + 1;
  const bool table = (size_t)2 * m.B * n_words <= lds_words;
  for (uint32_t x = tid; table && x < 2 * m.B * n_words; x += kOrdThreads) sm[x] = 0;
  const uint32_t edge_v[2] = {s_v[0], s_v[n_win - 1]}, edge_round[2] = {s_o[0] / kRound, s_o[n_win - 1] / kRound};
#pragma unroll
  for (uint32_t u = 0; u < kOrdPer; ++u) {
    const uint32_t r = u * kOrdThreads + tid;
    const bool head = r >= n_win || r == 0 || s_v[r - 1] != (v[u] & ~kRecKeeps) || s_o[r - 1] / kRound != o[u] / kRound;
    const uint64_t bits64 = __ballot(head);
    if ((tid & 63u) == 0) { heads[r >> 5] = (uint32_t)bits64; heads[(r >> 5) + 1] = (uint32_t)(bits64 >> 32); }
  }
  __syncthreads();
#pragma unroll
  for (uint32_t u = 0; u < kOrdPer; ++u) {
    const uint32_t r = u * kOrdThreads + tid;
    to[u] = r < n_win ? r : kNone;
    if (kSorted || r >= n_win) continue;
    // the group [from, end)
    const uint32_t upto = (2u << (r & 31)) - 1u;   // the bits up to r's
    uint32_t w = r >> 5, h = heads[w] & upto;
    while (!h) h = heads[--w];                      // (place 0 is a head)
    const uint32_t from = w * 32u + 31u - (uint32_t)__clz(h);
    w = r >> 5;
    h = heads[w] & ~upto;
    while (!h && w < kOrdWindow / 32) h = heads[++w];
    const uint32_t end = min(n_win, h ? w * 32u + (uint32_t)__ffs(h) - 1u : n_win);
    uint32_t smaller = 0, y = from;
    for (; y + 4 <= end; y += 4)
      smaller += (s_o[y] < o[u]) + (s_o[y + 1] < o[u]) + (s_o[y + 2] < o[u]) + (s_o[y + 3] < o[u]);
    for (; y < end; ++y) smaller += s_o[y] < o[u];
    to[u] = from + smaller;
    // (a group that stays in the margin may go on outside: its places are not looked at)
    const uint32_t crosses = (from == 0 && w_lo > 0 && end > x_lo - w_lo ? 1u : 0u) | (end == n_win && w_hi < m.O && from < s1 - w_lo ? 2u : 0u);
    if (crosses) atomicOr(&crossing, crosses);
  }
  __syncthreads();
  for (uint32_t side = 0; side < 2; ++side) {
    if (kSorted || !(crossing & (1u << side))) continue;   // the same for the whole workgroup
    // the group at this edge of the window goes on outside (it may also just end here)
    constexpr uint32_t kFar = kRound / kOrdThreads;
    uint32_t far_o[kFar], far_v[kFar], far_ifl[kFar], n_far = 0, n_near = 0;
    auto mark = [&](uint32_t x) { atomicOr(&bits[(x % kRound) >> 5], 1u << (x & 31)); };
    auto member = [&](uint32_t x, uint32_t rec_v) { return x != kNone && x / kRound == edge_round[side] && (rec_v & ~kRecKeeps) == edge_v[side]; };
#pragma unroll
    for (uint32_t u = 0; u < kFar; ++u) {
      const uint32_t d = u * kOrdThreads + tid;
      const bool in = side == 0 ? d < w_lo : d < m.O - w_hi;
      far_o[u] = in ? src[side == 0 ? w_lo - 1 - d : w_hi + d] : kNone;
      const uint64_t rec = in ? m.occ_rec[far_o[u]] : 0ull;
      far_v[u] = (uint32_t)rec;
      far_ifl[u] = (uint32_t)(rec >> 32);
      if (!member(far_o[u], far_v[u])) far_o[u] = kNone;
      if (far_o[u] != kNone) { ++n_far; mark(far_o[u]); }
    }
#pragma unroll
    for (uint32_t u = 0; u < kOrdPer; ++u)
      if (member(o[u], v[u])) { ++n_near; mark(o[u]); }
    const uint32_t mine = side == 0 ? n_far : n_near;
    if (mine) atomicAdd(&n_edge, mine);
    __syncthreads();
    const uint32_t first = side == 0 ? 0u - n_edge : n_win - n_edge;   // the group's first place (may wrap below zero)
    auto place = [&](uint32_t x) {
      const uint32_t word = (x % kRound) >> 5;
      uint32_t below = __popc(bits[word] & ((1u << (x & 31)) - 1u));
      for (uint32_t k = 0; k < word; ++k) below += __popc(bits[k]);
      return first + below;
    };
#pragma unroll
    for (uint32_t u = 0; u < kOrdPer; ++u)
      if (member(o[u], v[u])) to[u] = place(o[u]);
#pragma unroll
    for (uint32_t u = 0; u < kFar; ++u) {
      const uint32_t at = far_o[u] != kNone ? place(far_o[u]) : kNone;
      if (at < n_win) { s_o[at] = far_o[u] | (far_v[u] & kRecKeeps); s_ifl[at] = far_ifl[u]; }
    }
    __syncthreads();
    if (tid < kRound / 32) bits[tid] = 0;
    if (tid == 0) n_edge = 0;
    __syncthreads();
  }
#pragma unroll
  for (uint32_t u = 0; u < kOrdPer; ++u)
    if (to[u] < n_win) { s_o[to[u]] = o[u] | (v[u] & kRecKeeps); s_ifl[to[u]] = ifl[u]; }
  __syncthreads();
  constexpr uint32_t kOrdered = (kOrdBack + kOrdStretch + kOrdThreads - 1) / kOrdThreads;
  uint32_t blk[kOrdered];
  bool starts[kOrdered];
#pragma unroll
  for (uint32_t u = 0; u < kOrdered; ++u) {
    const uint32_t e = x_lo + u * kOrdThreads + tid;
    blk[u] = e < s1 ? m.instr_blk[s_ifl[e - w_lo] >> 2] : 0u;
  }
#pragma unroll
  for (uint32_t u = 0; u < kOrdered; ++u) {
    const uint32_t e = x_lo + u * kOrdThreads + tid;
    if (e < s1) s_blk[e - w_lo] = blk[u];
    starts[u] = e < s1 && m.blk_start[blk[u]] == s_ifl[e - w_lo] >> 2;
  }
  __syncthreads();
  uint32_t *const def_l = sm, *const use_l = sm + m.B * n_words;
#pragma unroll
  for (uint32_t u = 0; u < kOrdered; ++u) {
    const uint32_t e = x_lo + u * kOrdThreads + tid, r = e - w_lo;
    if (e < s0 || e >= s1) continue;
    const uint32_t ev = s_v[r], eo = s_o[r], ei = s_ifl[r];
    L.ent[e] = u32x4{eo & ~kRecKeeps, ei, ev | (eo & kRecKeeps) | (starts[u] ? kEntBlockStart : 0u), blk[u]};
    if (e == 0 || s_v[r - 1] != ev) L.first[ev] = eo & ~kRecKeeps;
    bool reads_first = false;   // is this mention group the first of its vreg in the block, and does it read?
    if (ei & VL_OCC_USE) {
      uint32_t x = r;   // (kOrdBack: the walk leaves the instruction before it leaves what is in order)
      while (x + w_lo > 0 && s_v[x - 1] == ev && (s_ifl[x - 1] >> 2) == (ei >> 2)) --x;
      reads_first = x + w_lo == 0 || s_v[x - 1] != ev || s_blk[x - 1] != blk[u];
    }
    const uint32_t bit = 1u << (ev & 31), at = blk[u] * n_words + (ev >> 5) - word0;
    if (table) {
      if (ei & VL_OCC_DEF) atomicOr(&def_l[at], bit);
      if (reads_first) atomicOr(&use_l[at], bit);
    } else {
      if (ei & VL_OCC_DEF) atomicOr(&L.def[(size_t)blk[u] * m.W + (ev >> 5)], bit);
      if (reads_first) atomicOr(&L.use[(size_t)blk[u] * m.W + (ev >> 5)], bit);
    }
  }
  if (!table) return;
  __syncthreads();
  // the first and the last word of the range may be shared with the neighbouring stretches
  for (uint32_t x = tid; x < m.B * n_words; x += kOrdThreads) {
    const size_t at = (size_t)(x / n_words) * m.W + word0 + x % n_words;
    if (def_l[x]) atomicOr(&L.def[at], def_l[x]);
    if (use_l[x]) atomicOr(&L.use[at], use_l[x]);
  }
}

// ---- 3. fixed point -------------------------------------------------------------------
// out[b] = OR of in[s] over successors; in[b] = use[b] | (out[b] & ~def[b]).  Bit columns
// do not interact, so each lane iterates its own word to its own fixed point; blocks are
// swept in reverse linear order.  LDS holds in/use/def of the wave's 64 words when the
// block count allows, otherwise the sweep runs on global memory.
template <bool kLds>
__global__ __launch_bounds__(64) void k_fixpoint(MIRS, const Grid grid) {
  const uint32_t prog = grid_prog(grid), bx = grid_block(grid);
  if (prog >= grid.n) return;
  const DevProg VL_CONSTANT &m = as_constant(mirs)[prog];
  const DevLive VL_CONSTANT &L = as_constant(lives)[prog];
  extern __shared__ uint32_t sm[];
  const uint32_t lane = threadIdx.x, w = bx * 64 + lane;
  if (bx * 64 >= m.W) return;
  const bool act = w < m.W;
  const uint32_t B = m.B, W = m.W;
  // in_l has one row more than there are blocks: row B stays empty and stands for "no successor"
  uint32_t *in_l = sm, *use_l = sm + (size_t)(B + 1) * 64, *def_l = use_l + (size_t)B * 64;
  // the successor lists are walked once per block and sweep: they sit in LDS too, and the
  // first two successors of each block (absent ones: row B) in arrays of their own
  uint32_t *succ_off_l = def_l + (size_t)B * 64, *succ_l = succ_off_l + B + 1;
  uint32_t *s0_l = succ_l + m.E, *s1_l = s0_l + B;
  if (kLds) {
    for (uint32_t x = lane; x <= B; x += 64) succ_off_l[x] = m.succ_off[x];
    for (uint32_t x = lane; x < m.E; x += 64) succ_l[x] = m.succ[x];
    for (uint32_t x = lane; x < B; x += 64) {
      const uint32_t e0 = m.succ_off[x], e1 = m.succ_off[x + 1];
      s0_l[x] = e0 < e1 ? m.succ[e0] : B;
      s1_l[x] = e0 + 1 < e1 ? m.succ[e0 + 1] : B;
    }
    in_l[B * 64 + lane] = 0;
    for (uint32_t b0 = 0; b0 < B; b0 += 8) {   // the rows of eight blocks in flight
      uint32_t uu[8], dd[8];
#pragma unroll
      for (uint32_t t = 0; t < 8; ++t) {
        const bool in = act && b0 + t < B;
        uu[t] = in ? L.use[(size_t)(b0 + t) * W + w] : 0;
        dd[t] = in ? L.def[(size_t)(b0 + t) * W + w] : 0;
      }
#pragma unroll
      for (uint32_t t = 0; t < 8; ++t)
        if (b0 + t < B) {
          in_l[(b0 + t) * 64 + lane] = 0;
          use_l[(b0 + t) * 64 + lane] = uu[t];
          def_l[(b0 + t) * 64 + lane] = dd[t];
        }
    }
  }
  uint32_t sweeps = 0;
  bool changed = true;
  while (kLds && __any(changed)) {   // monotone on a finite lattice: terminates
    // A block's step is: read the rows of its successors, combine, write its own row.  What
    // does not depend on the row just written (the successors' indices, use, def and the old
    // row of the next block) is fetched one block ahead.
    changed = false;
    ++sweeps;
    uint32_t s0 = s0_l[B - 1], s1 = s1_l[B - 1], u = use_l[(B - 1) * 64 + lane], d = def_l[(B - 1) * 64 + lane];
    uint32_t n_succ = succ_off_l[B] - succ_off_l[B - 1];
    for (uint32_t b = B; b-- > 0;) {
      uint32_t out = in_l[s0 * 64 + lane] | in_l[s1 * 64 + lane];
      const uint32_t old = in_l[b * 64 + lane];
      if (n_succ > 2)
        for (uint32_t e = succ_off_l[b] + 2; e < succ_off_l[b + 1]; ++e) out |= in_l[succ_l[e] * 64 + lane];
      const uint32_t nin = u | (out & ~d);
      if (b > 0) {
        s0 = s0_l[b - 1]; s1 = s1_l[b - 1];
        u = use_l[(b - 1) * 64 + lane]; d = def_l[(b - 1) * 64 + lane];
        n_succ = succ_off_l[b] - succ_off_l[b - 1];
      }
      if (nin != old) {
        changed = true;
        in_l[b * 64 + lane] = nin;
      }
    }
  }
  while (!kLds && __any(changed)) {
    changed = false;
    ++sweeps;
    for (uint32_t b = B; b-- > 0;) {
      uint32_t out = 0;
      const uint32_t e0 = kLds ? succ_off_l[b] : m.succ_off[b], e1 = kLds ? succ_off_l[b + 1] : m.succ_off[b + 1];
      for (uint32_t e = e0; e < e1; ++e) {
        uint32_t s = kLds ? succ_l[e] : m.succ[e];
        out |= kLds ? in_l[s * 64 + lane] : (act ? L.live_in[(size_t)s * W + w] : 0);
      }
      uint32_t u = kLds ? use_l[b * 64 + lane] : (act ? L.use[(size_t)b * W + w] : 0);
      uint32_t d = kLds ? def_l[b * 64 + lane] : (act ? L.def[(size_t)b * W + w] : 0);
      uint32_t nin = u | (out & ~d);
      uint32_t old = kLds ? in_l[b * 64 + lane] : (act ? L.live_in[(size_t)b * W + w] : 0);
      if (nin != old) {
        changed = true;
        if (kLds) in_l[b * 64 + lane] = nin; else if (act) L.live_in[(size_t)b * W + w] = nin;
      }
    }
  }
  // write-out: in (when it lived in LDS) and out
  if (kLds) {
#pragma unroll 4
    for (uint32_t b = 0; b < B; ++b) {
      uint32_t out = in_l[s0_l[b] * 64 + lane] | in_l[s1_l[b] * 64 + lane];
      if (succ_off_l[b + 1] - succ_off_l[b] > 2)
        for (uint32_t e = succ_off_l[b] + 2; e < succ_off_l[b + 1]; ++e) out |= in_l[succ_l[e] * 64 + lane];
      if (act) {
        L.live_out[(size_t)b * W + w] = out;
        L.live_in[(size_t)b * W + w] = in_l[b * 64 + lane];
      }
    }
  }
  for (uint32_t b = 0; !kLds && b < B; ++b) {
    uint32_t out = 0;
    const uint32_t e0 = kLds ? succ_off_l[b] : m.succ_off[b], e1 = kLds ? succ_off_l[b + 1] : m.succ_off[b + 1];
    for (uint32_t e = e0; e < e1; ++e) {
      uint32_t s = kLds ? succ_l[e] : m.succ[e];
      out |= kLds ? in_l[s * 64 + lane] : (act ? L.live_in[(size_t)s * W + w] : 0);
    }
    if (act) {
      L.live_out[(size_t)b * W + w] = out;
      if (kLds) L.live_in[(size_t)b * W + w] = in_l[b * 64 + lane];
    }
  }
  // last block each vreg is live into (0 when there is none after the entry): lets the interval
  // kernels stop looking at later blocks.  Blocks in descending order; a lane owns its 32 vregs.
  uint32_t seen = 0;
  for (uint32_t b = B; b-- > 1;) {
    const uint32_t in_b = kLds ? in_l[b * 64 + lane] : (act ? L.live_in[(size_t)b * W + w] : 0);
    uint32_t fresh = in_b & ~seen;
    seen |= in_b;
    while (act && fresh) {
      const uint32_t v = w * 32 + __ffs(fresh) - 1;
      fresh &= fresh - 1;
      if (v < m.V) L.last_live[v] = b;
    }
  }
  uint32_t in0 = kLds ? in_l[lane] : (act ? L.live_in[w] : 0);
  if (act && in0) L.counters[kCtrNotStrict] = 1;
  if (lane == 0) atomicMax(&L.counters[kCtrSweeps], sweeps);
}

// Up to 32 blocks (every shape of loop nest that the benchmark's programs have): the rows of a
// wavefront's 64 words stay in registers, a lane holding its word of every block.  What bounds the
// sweeps is the chain from block to block (read the successors' rows, combine, write): a row that
// is picked by a scalar index costs a few cycles there, a row in LDS two trips of a hundred.  The
// last live block of each vreg is collected as five bit planes over the lane's 32 vregs and written
// a vector of four at a time, where a loop over the set bits of every block's row stored them one by one.
// (8,000 instructions in 22 blocks: 21.6 us through LDS, 9.5 this way; 256 of 1,000-20,000: 34 and 19.)
constexpr uint32_t kRegBlocks = 32;
__global__ __launch_bounds__(64) void k_fixpoint_regs(MIRS, const Grid grid) {
  const uint32_t prog = grid_prog(grid), bx = grid_block(grid);
  if (prog >= grid.n) return;
  const DevProg VL_CONSTANT &m = as_constant(mirs)[prog];
  const DevLive VL_CONSTANT &L = as_constant(lives)[prog];
  const uint32_t lane = threadIdx.x, w = bx * 64 + lane;
  const uint32_t B = m.B, W = m.W;
  if (bx * 64 >= W) return;
  const bool act = w < W;
  const uint32_t col = min(w, W - 1);
  typedef uint32_t rows_t __attribute__((ext_vector_type(kRegBlocks)));   // (a vector, so that a scalar index stays in registers)
  rows_t in = 0, use, def;
  // lane b: the first two successors of block b (one: twice; none: marked), and whether there are more
  constexpr uint32_t kNoSucc = 1u << 16, kMoreSucc = 1u << 17;
  uint32_t succ = kNoSucc;
  if (lane < B) {
    const uint32_t e0 = m.succ_off[lane], n = m.succ_off[lane + 1] - e0;
    if (n) {
      const uint32_t s0 = m.succ[e0], s1 = m.succ[e0 + (n > 1 ? 1 : 0)];
      succ = s0 | (s1 << 8) | (n > 2 ? kMoreSucc : 0u);
    }
  }
  const __amdgpu_buffer_rsrc_t use_rows = __builtin_amdgcn_make_buffer_rsrc((void *)(uintptr_t)L.use, 0, B * W * 4, 0x00020000);
  const __amdgpu_buffer_rsrc_t def_rows = __builtin_amdgcn_make_buffer_rsrc((void *)(uintptr_t)L.def, 0, B * W * 4, 0x00020000);
#pragma unroll
  for (uint32_t b = 0; b < kRegBlocks; ++b) {   // all in flight; what lies beyond the last row reads as zero (and is not looked at)
    use[b] = __builtin_amdgcn_raw_buffer_load_b32(use_rows, (col + b * W) * 4, 0, 0);
    def[b] = __builtin_amdgcn_raw_buffer_load_b32(def_rows, (col + b * W) * 4, 0, 0);
  }
  auto out_of = [&](uint32_t b) __attribute__((always_inline)) {
    const uint32_t s = __builtin_amdgcn_readlane(succ, b);
    uint32_t out = in[s & 31u] | in[(s >> 8) & 31u];
    if (s & (kNoSucc | kMoreSucc)) {
      if (s & kNoSucc) out = 0;
      else
        for (uint32_t e = m.succ_off[b] + 2; e < m.succ_off[b + 1]; ++e) out |= in[m.succ[e] & 31u];
    }
    return out;
  };
  // (the loops over blocks stay loops: spelt out, the code is 40 KB that every launch fetches anew)
  uint32_t sweeps = 0, changed;
  do {   // monotone on a finite lattice: terminates
    changed = 0;
    ++sweeps;
#pragma unroll 1
    for (uint32_t b = B; b-- > 0;) {
      const uint32_t now = use[b] | (out_of(b) & ~def[b]);
      changed |= now ^ in[b];
      in[b] = now;
    }
  } while (__any(changed != 0));
  uint32_t seen = 0, plane[5] = {};
#pragma unroll 1
  for (uint32_t b = B; b-- > 0;) {
    const uint32_t out = out_of(b), now = in[b], fresh = now & ~seen;
    if (act) {
      L.live_out[(size_t)b * W + w] = out;
      L.live_in[(size_t)b * W + w] = now;
    }
    seen |= fresh;
#pragma unroll
    for (uint32_t j = 0; j < 5; ++j) plane[j] |= (b >> j) & 1u ? fresh : 0u;
  }
  if (act) {   // (the array is a whole number of 256-byte vectors long: it has room for the last word's 32)
    u32x4 VL_GLOBAL *to = reinterpret_cast<u32x4 VL_GLOBAL *>(L.last_live + (size_t)w * 32);
#pragma unroll
    for (uint32_t v = 0; v < 32; v += 4) {
      u32x4 x = 0;
#pragma unroll
      for (uint32_t t = 0; t < 4; ++t)
#pragma unroll
        for (uint32_t j = 0; j < 5; ++j) x[t] |= ((plane[j] >> (v + t)) & 1u) << j;
      to[v / 4] = x;
    }
    if (in[0]) L.counters[kCtrNotStrict] = 1;
  }
  if (lane == 0) atomicMax(&L.counters[kCtrSweeps], sweeps);
}

// one-byte summary of where membership in P(.) changes inside a mention group's stretch
constexpr uint8_t kStartI = 1, kStartI1 = 2, kEndI = 4, kEndI1 = 8, kEndN = 16, kAgain = 32, kOpenBefore = 64;

// exclusive prefixes over a workgroup of kStretch threads, of n values per thread at once: x[k] of all threads,
// the total of which goes to sums[k] (those from n_sums on are dropped)
template <uint32_t n>
__device__ inline void stretch_prefix(uint32_t (&x)[n], uint32_t VL_GLOBAL *sums, uint32_t n_sums) {
  __shared__ uint32_t part[n][kStretch / 64];
  const uint32_t wave = threadIdx.x >> 6;
  uint32_t incl[n];
#pragma unroll
  for (uint32_t k = 0; k < n; ++k) {
    incl[k] = wave_prefix(x[k]);
    if ((threadIdx.x & 63u) == 63u) part[k][wave] = incl[k];
  }
  __syncthreads();
#pragma unroll
  for (uint32_t k = 0; k < n; ++k) {
    uint32_t before = 0, total = 0;
#pragma unroll
    for (uint32_t y = 0; y < kStretch / 64; ++y) {
      before += y < wave ? part[k][y] : 0u;
      total += part[k][y];
    }
    if (threadIdx.x == k && k < n_sums) sums[k] = total;
    x[k] = before + incl[k] - x[k];
  }
}

// ---- 4. per-occurrence liveness, kill flags and event roles ---------------------------
// For the mentions of v at instruction i (its "group"): v is live after i iff the next
// mention of v in the same block reads it, or, with no later mention in the block, v is
// in the block's live-out.  P(i) contains v iff it is live after i or written at i.
constexpr uint32_t kEvtThreads = 256, kEvtHalo = 16, kEvtWindow = kEvtThreads + 2 * kEvtHalo;

// (One-dimensional grid: block_map names the kernel and the stretch of 256 entries of every
// workgroup, so that no workgroup is launched for stretches a smaller kernel does not have.)
__global__ __launch_bounds__(kEvtThreads) void k_events(MIRS, const uint2 *__restrict__ block_map) {
  const uint2 where = block_map ? block_map[blockIdx.x] : make_uint2(0, blockIdx.x);
  if (where.x == kNone) return;   // (a die with fewer blocks than the others)
  const DevProg VL_CONSTANT &m = as_constant(mirs)[where.x];
  const DevLive VL_CONSTANT &L = as_constant(lives)[where.x];
  // The neighbours of an entry in the sorted order (its own mention group, the groups before
  // and after it) are looked at many times: the workgroup's stretch of entries plus a halo
  // on both sides is staged in LDS once, and only what lies beyond the halo is read from
  // memory.
  __shared__ u32x4 s_ent[kEvtWindow];
  const uint32_t base = where.y * kEvtThreads;
  if (base >= m.O) return;
  const uint32_t win_lo = base - kEvtHalo;   // may wrap below zero: window indices are taken modulo 2^32
  for (uint32_t r = threadIdx.x; r < kEvtWindow; r += kEvtThreads) {
    const uint32_t x = win_lo + r;
    const bool in = x < m.O;   // false for the wrapped indices too
    s_ent[r] = in ? L.ent[x] : u32x4{0u, 0u, kNone, 0u};
  }
  __syncthreads();
  const uint32_t e = base + threadIdx.x;
  // (the part below leaves early where an entry has nothing to count)
  auto count_runs = [&]() __attribute__((always_inline)) -> uint32_t {
  if (e >= m.O) return 0;
  auto ent = [&](uint32_t x) { const uint32_t r = x - win_lo; return r < kEvtWindow ? s_ent[r].y : L.ent[x].y; };
  auto occ_at = [&](uint32_t x) { const uint32_t r = x - win_lo; return r < kEvtWindow ? s_ent[r].x : L.ent[x].x; };
  auto kept_at = [&](uint32_t x) { const uint32_t r = x - win_lo; return ((r < kEvtWindow ? s_ent[r].z : L.ent[x].z) & kRecKeeps) != 0; };
  auto blk_at = [&](uint32_t x) { const uint32_t r = x - win_lo; return r < kEvtWindow ? s_ent[r].w : L.ent[x].w; };
  const u32x4 own = s_ent[threadIdx.x + kEvtHalo];
  const uint32_t o = own.x, v = own.z & kEntVreg, ifl = own.y, i = ifl >> 2;
  // What is read from memory depends on (v, i) first and on the blocks found second: the reads
  // of each level are issued together, with indices clamped where the value may not be needed,
  // so that a lane waits for memory twice instead of once per branch taken.
  const uint32_t lo = L.vcnt[v], hi = L.vcnt[v + 1];
  const uint32_t b = own.w;
  const bool keeps = (own.z & kRecKeeps) != 0, at_start = (own.z & kEntBlockStart) != 0;
  const uint32_t attr = m.vattr[v], last_live_v = L.last_live[v];
  uint32_t gs = e, ge = e + 1;
  while (gs > lo && (ent(gs - 1) >> 2) == i) --gs;
  while (ge < hi && (ent(ge) >> 2) == i) ++ge;
  bool has_use = false, has_def = false;
  uint32_t first_use = kNone, first_def = kNone;
  for (uint32_t x = gs; x < ge; ++x) {
    const uint32_t f = x == e ? ifl : ent(x);
    if (f & VL_OCC_USE) { has_use = true; if (first_use == kNone) first_use = x; }
    if (f & VL_OCC_DEF) { has_def = true; if (first_def == kNone) first_def = x; }
  }
  const uint32_t nxt = ge < hi ? ent(ge) : 0u;
  // second level
  const uint32_t vw = v >> 5, vbit = 1u << (v & 31);
  const uint32_t blk_next = ge < hi ? blk_at(ge) : 0u;
  const bool out_b = (L.live_out[(size_t)b * m.W + vw] & vbit) != 0;
  const bool out_below = (L.live_out[(size_t)(b > 0 ? b - 1 : 0) * m.W + vw] & vbit) != 0;
  const uint32_t start_b = m.blk_start[b], start_b1 = m.blk_start[b + 1], start_b2 = m.blk_start[min(b + 2, m.B)];
  const bool in_after = (L.live_in[(size_t)min(b + 1, m.B - 1) * m.W + vw] & vbit) != 0;   // live into the block after b
  const uint32_t F = m.class_size[attr_class(attr)];
  bool la;
  if (ge < hi && blk_next == b) {
    la = (nxt & VL_OCC_USE) != 0;
    for (uint32_t x = ge + 1; x < hi && (ent(x) >> 2) == (nxt >> 2); ++x) la |= (ent(x) & VL_OCC_USE) != 0;
  } else {
    la = out_b;
  }
  const uint32_t fl = ifl & 3u;
  const bool kill = (fl & VL_OCC_USE) && !has_def && !la;
  uint8_t role = 0;
  // an instruction with an early-clobber definition keeps what it reads occupied until it has
  // written: the operand that dies here is released after the definitions have been tested
  if (!has_def && !la && e == first_use) role |= keeps ? kRolePostKill : kRolePreKill;
  if (has_def && e == first_def) {
    if (!has_use) role |= kRoleTestSet;
    if (!la) role |= kRolePostKill;
  }
  if (e == lo) role |= kRoleFirst;
  L.occ_role[o] = role | (kill ? kRoleKill : 0);
  const uint32_t prev = e > lo ? occ_at(e - 1) : kNone;
  if (prev != kNone && o - prev >= 0xFFFFu) L.prev_occ[o] = prev;
  // the occurrence's check record (its events are counted per instruction by a later pass over the roles)
  {
    // when an occurrence is checked the ring ends with that occurrence's chunk
    const uint32_t next = e + 1 < hi ? occ_at(e + 1) : o;
    const bool keep = o + kWalkReach < (next / kWalkChunk + 1u) * kWalkChunk && next - o <= kKeepMaxGap;
    const uint32_t delta = prev == kNone ? 0u : min(o - prev, 0xFFFFu);
    const bool near = prev != kNone && delta != 0xFFFFu && check_reaches(o, prev);
    const uint32_t width = attr_width(attr), align = attr_align(attr);
    const bool is_first = (role & kRoleFirst) != 0;
    const bool generic = is_first && ((align & (align - 1u)) != 0 || m.has_reserved || width > F);
    const bool simple = is_first && !generic;
    u32x4 r;
    r.x = (is_first ? kPlanFirst : kPlanChk) | (keep ? kPlanKeep : 0u) | (near ? kChkNear : 0u) | (generic ? kChkGeneric : 0u) |
          ((o % kWalkRing) << 8) | (((near ? prev : o) % kWalkRing) << 20);
    r.y = delta | (attr << 16);
    r.z = simple ? (align - 1u) * 0x10001u : 0u;
    r.w = simple ? min(F - width, 0xFFFFu) * 0x10001u : 0xFFFFFFFFu;
    L.chk[o] = r;
  }
  L.ent_info[e] = (uint8_t)((la ? kEntLiveAfter : 0) | (has_use ? kEntHasUse : 0) | (has_def ? kEntHasDef : 0) |
                            (e == gs ? kEntGroupStart : 0) | (keeps && has_use ? kEntKept : 0));

  // ---- live intervals, counting pass (the filling pass and the reasoning are at f_seg) ----
  // The first entry of each mention group owns the stretch from i up to the next mention of v
  // and counts the run starts in it; what the neighbouring groups contribute is worked out
  // from their flags here, since their own threads may not have run yet.
  if (e != gs) { L.ent_sf[e] = 0; return 0; }
  bool cur;   // was v occupied just before this stretch?
  if (i == 0) cur = false;
  else if (gs > lo && (ent(gs - 1) >> 2) == i - 1) {
    bool prev_def = false, prev_kept_use = false;
    for (uint32_t x = gs; x-- > lo && (ent(x) >> 2) == i - 1;) {
      prev_def |= (ent(x) & VL_OCC_DEF) != 0;
      prev_kept_use |= (ent(x) & VL_OCC_USE) != 0 && kept_at(x);
    }
    // live after i - 1: this group is the next mention; in another block (the one below) the
    // block's live-out decides
    cur = prev_def || (at_start ? out_below : has_use) || prev_kept_use;
  } else if (i > start_b) cur = has_use;
  else cur = out_below;
  uint8_t sf = cur ? kOpenBefore : 0;
  uint32_t n_start = 0;
  auto span = [&](uint32_t s, uint32_t t, bool member) {
    if (t <= s) return;
    if (member && !cur) {
      ++n_start;
      sf |= s == i ? kStartI : s == i + 1 ? kStartI1 : kAgain;
    }
    if (!member && cur) sf |= s == i ? kEndI : s == i + 1 ? kEndI1 : kAgain;
    cur = member;
  };
  span(i, i + 1, has_def || la || (keeps && has_use));
  const uint32_t i2 = ge < hi ? nxt >> 2 : m.N;
  const uint32_t b2 = ge < hi ? blk_next : m.B;
  const uint32_t start_next = m.blk_start[b2];   // third level; only needed when the next mention is in another block
  if (b2 == b) {
    span(i + 1, i2, la);
  } else {
    span(i + 1, start_b1, la);
    // blocks in between: v is live into none of them after its last live block.  The block
    // right after b (nearly always the only one) was read with the second level.
    const uint32_t xe = min(b2, max(b + 1, last_live_v + 1));
    if (b + 1 < xe) span(start_b1, start_b2, in_after);
    for (uint32_t x = b + 2; x < xe; ++x)
      span(m.blk_start[x], m.blk_start[x + 1], bit_get(L.live_in + (size_t)x * m.W, v));
    if (xe < b2) {
      if (xe == b + 1) span(start_b1, start_b2, false);
      else span(m.blk_start[xe], m.blk_start[xe + 1], false);
    }
    if (ge < hi) {
      bool next_use = false;
      for (uint32_t x = ge; x < hi && (ent(x) >> 2) == i2; ++x) next_use |= (ent(x) & VL_OCC_USE) != 0;
      span(start_next, i2, next_use);
    }
  }
  if (ge >= hi && cur) sf |= kEndN;
  if (n_start > 1) sf |= kAgain;   // two starts in one stretch cannot be told apart by the summary
  L.ent_sf[e] = sf;
  return n_start;
  };
  // where the runs of each entry go, from the stretch's first
  uint32_t runs[1] = {count_runs()};
  stretch_prefix(runs, L.seg_base + where.y, 1);
  if (e < m.O) L.ent_seg[e] = runs[0];
}

// The grids are sized for the largest kernel of the batch, so most blocks belong to smaller
// kernels and exit at once.  A block of the part that counts each instruction's events (light
// work) takes this many stretches of 256 instructions, which keeps their number down; the
// heavier parts are faster with one stretch per block.
constexpr uint32_t kStageReps = 4;

// ---- 5a. event stream -----------------------------------------------------------------
__device__ inline uint32_t item_of_instr(const DevProg VL_CONSTANT &m, uint32_t i) { return i + m.instr_blk[i] + 1; }

__device__ inline uint32_t wave_incl_scan(uint32_t x) {
  for (int d = 1; d < 64; d <<= 1) {
    uint32_t y = __shfl_up(x, d, 64);
    if ((int)(threadIdx.x & 63) >= d) x += y;
  }
  return x;
}

// nearest occurrence of v before instruction `at`, else the first at or after it
__device__ inline uint32_t source_occurrence(const DevLive VL_CONSTANT &L, uint32_t v, uint32_t at) {
  const uint32_t lo = L.vcnt[v], hi = L.vcnt[v + 1];
  const uint32_t x = first_entry_at(L, lo, hi, at);
  return x > lo ? L.ent[x - 1].x : (x < hi ? L.ent[x].x : 0u);
}

// The record of one occupancy event (layout in vl_dev.h).  `near`: the occurrence is
// certainly inside the verifier's ring when the event is replayed.
__device__ inline u32x4 event_record(uint32_t o, uint32_t v, uint32_t attr, bool tested, bool near) {
  const uint32_t width = attr_width(attr);
  const bool slow = !near || attr_straddle(attr) || width == 32;
  u32x4 r;
  r.x = (o % kWalkRing) | (v << 8);
  r.y = width == 32 ? 0xFFFFFFFFu : ((1u << width) - 1u);
  r.z = attr_word(attr) * 256u;
  r.w = o | (slow ? kEvtSlow : 0u) | (tested ? kEvtTested : 0u);
  return r;
}
__device__ inline u32x4 event_record(const DevProg VL_CONSTANT &m, uint32_t o, uint32_t v, bool tested, bool near) {
  return event_record(o, v, m.vattr[v], tested, near);
}

// Between two blocks adjacent in the linear order the occupied set changes from the
// earlier block's live-out to the later block's live-in: one wave per boundary lists the
// values that leave (release) and those that enter (occupy without test).
template <bool kFill>
__device__ inline void f_boundary(const DevProg VL_CONSTANT &m, const DevLive VL_CONSTANT &L, const uint32_t bx, const uint32_t tx,
                                  const uint32_t bdim) {
  const uint32_t b = bx, lane = tx;
  if (b >= m.B) return;
  const uint32_t item = m.blk_start[b] + b;
  if (b == 0) {
    if (!kFill && lane == 0) L.bound_off[0] = 0;
    return;
  }
  const uint32_t W = m.W, at = m.blk_start[b];
  const uint32_t VL_GLOBAL *out_prev = L.live_out + (size_t)(b - 1) * W;
  const uint32_t VL_GLOBAL *in_cur = L.live_in + (size_t)b * W;
  uint32_t base = kFill ? L.item_off[item] : 0, total = 0;
  // Filling: a lane first lists the vregs of its word in LDS; then the wavefront completes
  // one record per lane, so that the look-ups of the source occurrences run side by side.
  constexpr uint32_t kList = 512;
  __shared__ uint32_t s_list[kFill ? 4 * kList : 1];
  uint32_t *list = s_list + (kFill ? (threadIdx.x >> 6) * kList : 0);
  auto record = [&](uint32_t v) {
    const uint32_t src = source_occurrence(L, v, at);
    // replayed with the block's first instruction, when the readable window ends at
    // most 127 occurrences after that instruction's first operand
    const bool near = src < m.occ_off[at] && src + (kWalkReach - 2 * kWalkChunk + 1) >= m.occ_off[at];
    return event_record(m, src, v, false, near);
  };
  if (!kFill) {   // counting needs no positions: both directions at once, one reduction at the end
    uint32_t mine = 0;
    for (uint32_t w = lane; w < W; w += 64) mine += __popc(out_prev[w] ^ in_cur[w]);
    for (int d = 32; d >= 1; d >>= 1) mine += (uint32_t)__shfl_xor((int)mine, d, 64);
    if (lane == 0) L.bound_off[b] = mine;
    return;
  }
  for (int pass = 0; pass < 2; ++pass) {  // 0: leaving, 1: entering
    for (uint32_t w0 = 0; w0 < W; w0 += 64) {
      const uint32_t w = w0 + lane;
      uint32_t bits = 0;
      if (w < W) bits = pass == 0 ? (out_prev[w] & ~in_cur[w]) : (in_cur[w] & ~out_prev[w]);
      const uint32_t c = __popc(bits), incl = wave_incl_scan(c);
      const uint32_t n_here = __shfl(incl, 63, 64);
      if (kFill && n_here) {
        uint32_t pos = incl - c;
        const bool listed = n_here <= kList;   // the same in every lane
        while (bits) {
          const uint32_t v = w * 32 + __ffs(bits) - 1;
          bits &= bits - 1;
          if (listed) list[pos++] = v;
          else L.plan[base + total + pos++] = record(v);
        }
        if (listed) {
          __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
          __builtin_amdgcn_wave_barrier();
          for (uint32_t x = lane; x < n_here; x += 64) L.plan[base + total + x] = record(list[x]);
          __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
          __builtin_amdgcn_wave_barrier();
        }
      }
      total += n_here;
    }
  }
}

// Occupancy events of each instruction, in the order they take effect: releases of
// operands that die here, then test-and-occupy of the values written, then releases of
// values that are dead once the instruction has executed.
__device__ inline void f_plan_fill(const DevProg VL_CONSTANT &m, const DevLive VL_CONSTANT &L, const uint32_t bx, const uint32_t tx,
                                   const uint32_t bdim) {
  uint32_t i = bx * bdim + tx;
  if (i >= m.N) return;
  // the instruction's first event: those of earlier stretches, of earlier instructions in its own, and of block boundaries
  const uint32_t blk = m.instr_blk[i], item = i + blk + 1, in_order = L.item_base[bx] + L.item_off[item];
  const uint32_t base = in_order + L.bound_off[blk + 1];
  L.item_off[item] = base;
  uint32_t first = base;   // a block boundary's events go with the block's first instruction
  if (m.blk_start[blk] == i) L.item_off[item - 1] = first = in_order + L.bound_off[blk];
  const uint32_t o0 = m.occ_off[i], o1 = m.occ_off[i + 1];
  // evt_cut[c]: the first event of the instruction that occurrence 64 c belongs to (its events may be
  // replayed once the occurrences before 64 (c + 1) are staged); no instruction has more than 64
  static_assert(kMaxOperands <= kWalkChunk, "an instruction holds the first occurrence of one chunk at most");
  const uint32_t chunk = (o0 + kWalkChunk - 1) / kWalkChunk;
  if (chunk * kWalkChunk < o1) L.evt_cut[chunk] = first;
  if (i + 1 == m.N) {
    const uint32_t all = L.item_base[stretches(m.N)] + L.bound_off[m.B];
    L.item_off[item + 1] = all;
    L.evt_cut[(m.O + kWalkChunk - 1) / kWalkChunk] = all;
  }
  uint32_t n_pre = 0, n_set = 0;
  if (o1 - o0 <= 4) {
    // the common case: roles and vregs of all operands are read together, then their
    // attributes, so that the lane waits once per level instead of once per operand
    const uint32_t n = o1 - o0;
    uint32_t role[4], vv[4], aa[4];
#pragma unroll
    for (uint32_t u = 0; u < 4; ++u) {
      role[u] = u < n ? (uint32_t)L.occ_role[o0 + u] : 0u;
      vv[u] = u < n ? m.occ_vreg[o0 + u] : 0u;
    }
#pragma unroll
    for (uint32_t u = 0; u < 4; ++u) aa[u] = m.vattr[vv[u]];
#pragma unroll
    for (uint32_t u = 0; u < 4; ++u) {
      if (u < n) L.occ_kill[o0 + u] = (role[u] & kRoleKill) ? 1 : 0;
      n_pre += (role[u] & kRolePreKill) ? 1u : 0u;
      n_set += (role[u] & kRoleTestSet) ? 1u : 0u;
    }
    uint32_t at_pre = base, at_set = base + n_pre, at_post = base + n_pre + n_set;
#pragma unroll
    for (uint32_t u = 0; u < 4; ++u) {
      if (!(role[u] & (kRolePreKill | kRoleTestSet | kRolePostKill))) continue;
      const u32x4 r = event_record(o0 + u, vv[u], aa[u], false, true);
      if (role[u] & kRolePreKill) L.plan[at_pre++] = r;
      if (role[u] & kRoleTestSet) { u32x4 q = r; q.w |= kEvtTested; L.plan[at_set++] = q; }
      if (role[u] & kRolePostKill) { u32x4 q = r; q.w |= kEvtPost; L.plan[at_post++] = q; }
    }
    return;
  }
  for (uint32_t o = o0; o < o1; ++o) {
    const uint32_t role = L.occ_role[o];
    L.occ_kill[o] = (role & kRoleKill) ? 1 : 0;   // kill flags, in occurrence order
    n_pre += (role & kRolePreKill) ? 1u : 0u;
    n_set += (role & kRoleTestSet) ? 1u : 0u;
  }
  uint32_t at_pre = base, at_set = base + n_pre, at_post = base + n_pre + n_set;
  for (uint32_t o = o0; o < o1; ++o) {
    const uint32_t role = L.occ_role[o];
    if (!(role & (kRolePreKill | kRoleTestSet | kRolePostKill))) continue;
    // an instruction's own operands are always inside the ring when its events are replayed
    const u32x4 r = event_record(m, o, m.occ_vreg[o], false, true);
    if (role & kRolePreKill) L.plan[at_pre++] = r;
    if (role & kRoleTestSet) { u32x4 q = r; q.w |= kEvtTested; L.plan[at_set++] = q; }
    if (role & kRolePostKill) { u32x4 q = r; q.w |= kEvtPost; L.plan[at_post++] = q; }
  }
}

// Number of events of each instruction (the roles of its operands, as the filling pass above has
// them), prefixed over its stretch; kStageReps stretches at a time, side by side.
__device__ inline void f_item_count(const DevProg VL_CONSTANT &m, const DevLive VL_CONSTANT &L, const uint32_t bx, const uint32_t tx) {
  const uint32_t s0 = bx * kStageReps, n_stretch = stretches(m.N);
  if (s0 >= n_stretch) return;
  uint32_t o0[kStageReps], n_op[kStageReps], blk[kStageReps], n_evt[kStageReps], role[kStageReps][4];
#pragma unroll
  for (uint32_t r = 0; r < kStageReps; ++r) {
    const uint32_t i = (s0 + r) * kStretch + tx;
    o0[r] = i < m.N ? m.occ_off[i] : 0u;
    n_op[r] = i < m.N ? m.occ_off[i + 1] - o0[r] : 0u;
    blk[r] = i < m.N ? m.instr_blk[i] : 0u;
  }
#pragma unroll
  for (uint32_t r = 0; r < kStageReps; ++r)
#pragma unroll
    for (uint32_t u = 0; u < 4; ++u) role[r][u] = u < n_op[r] ? (uint32_t)L.occ_role[o0[r] + u] : 0u;
  constexpr uint32_t kEvents = kRolePreKill | kRoleTestSet | kRolePostKill;
#pragma unroll
  for (uint32_t r = 0; r < kStageReps; ++r) {
    n_evt[r] = 0;
#pragma unroll
    for (uint32_t u = 0; u < 4; ++u) n_evt[r] += __popc(role[r][u] & kEvents);
    for (uint32_t u = 4; u < n_op[r]; ++u) n_evt[r] += __popc(L.occ_role[o0[r] + u] & kEvents);
  }
  stretch_prefix(n_evt, L.item_base + s0, n_stretch - s0);
#pragma unroll
  for (uint32_t r = 0; r < kStageReps; ++r) {
    const uint32_t i = (s0 + r) * kStretch + tx;
    if (i < m.N) L.item_off[i + blk[r] + 1] = n_evt[r];
  }
}

// ---- 5b. live intervals ---------------------------------------------------------------
// Membership of v in P(.) changes only at instructions that mention v and at block
// boundaries.  The lane of each mention group (all mentions of v at one instruction) owns
// the stretch from its instruction up to the next mention of v (the last group: up to the
// end of the program) and finds the run starts and ends inside it; what holds just before
// the stretch is known locally.  Groups are sorted by (vreg, instruction), so a prefix sum
// of the start counts numbers the runs in CSR order; the j-th end belongs to the j-th start.
__device__ inline void f_seg_fill(const DevProg VL_CONSTANT &m, const DevLive VL_CONSTANT &L, const uint32_t bx, const uint32_t tx,
                                  const uint32_t bdim) {
  const uint32_t e = bx * bdim + tx;
  if (e >= m.O) return;
  // The counting pass (in the per-occurrence kernel) left a one-byte summary per entry.
  // Nearly every stretch changes membership only at its own instruction i, at i + 1 or at
  // the end of the program, and then the summary says everything needed here; the other
  // stretches (those with changes at block boundaries) are worked out again.
  const uint8_t sf = L.ent_sf[e];
  if (!(sf & (kStartI | kStartI1 | kEndI | kEndI1 | kEndN | kAgain))) return;
  const uint32_t i = L.ent[e].y >> 2;
  // runs that started before this stretch and ended before it: the end index lags the
  // start index by one exactly while a run is open
  size_t n_start = L.seg_base[bx] + L.ent_seg[e];
  size_t n_end = n_start - ((sf & kOpenBefore) ? 1u : 0u);
  if (!(sf & kAgain)) {
    if (sf & kStartI) L.seg[2 * n_start] = i;
    if (sf & kStartI1) L.seg[2 * n_start] = i + 1;
    if (sf & kEndI) L.seg[2 * n_end++ + 1] = i;
    if (sf & kEndI1) L.seg[2 * n_end++ + 1] = i + 1;
    if (sf & kEndN) L.seg[2 * n_end + 1] = m.N;
    return;
  }
  const uint8_t info = L.ent_info[e];
  const uint32_t v = L.ent[e].z & kEntVreg;
  const uint32_t hi = L.vcnt[v + 1], b = m.instr_blk[i];
  bool cur = (sf & kOpenBefore) != 0;
  auto span = [&](uint32_t s, uint32_t t, bool member) {
    if (t <= s) return;
    if (member && !cur) L.seg[2 * n_start++] = s;
    if (!member && cur) L.seg[2 * n_end++ + 1] = s;
    cur = member;
  };
  uint32_t ge = e + 1;
  while (ge < hi && (L.ent[ge].y >> 2) == i) ++ge;
  const bool la = (info & kEntLiveAfter) != 0;
  span(i, i + 1, (info & (kEntHasDef | kEntKept)) || la);
  const uint32_t i2 = ge < hi ? L.ent[ge].y >> 2 : m.N;
  const uint32_t b2 = ge < hi ? m.instr_blk[i2] : m.B;
  if (b2 == b) {
    span(i + 1, i2, la);
  } else {
    span(i + 1, m.blk_start[b + 1], la);
    const uint32_t xe = min(b2, max(b + 1, L.last_live[v] + 1));
    for (uint32_t x = b + 1; x < xe; ++x)
      span(m.blk_start[x], m.blk_start[x + 1], bit_get(L.live_in + (size_t)x * m.W, v));
    if (xe < b2) span(m.blk_start[xe], m.blk_start[xe + 1], false);
    if (ge < hi) span(m.blk_start[b2], i2, (L.ent_info[ge] & kEntHasUse) != 0);
  }
  if (ge >= hi && cur) L.seg[2 * n_end + 1] = m.N;
}

// where each vreg's (ascending) runs begin, and its hull: [first start, last end), or [0,0) without runs
__device__ inline void f_hull(const DevProg VL_CONSTANT &m, const DevLive VL_CONSTANT &L, const uint32_t bx, const uint32_t tx,
                              const uint32_t bdim) {
  const uint32_t v = bx * bdim + tx;
  if (v > m.V) return;
  auto runs_before = [&](uint32_t e) { return e < m.O ? L.seg_base[e / kStretch] + L.ent_seg[e] : L.seg_base[stretches(m.O)]; };
  const uint32_t s0 = runs_before(L.vcnt[v]);
  L.seg_off[v] = s0;
  if (v == m.V) return;
  const uint32_t s1 = runs_before(L.vcnt[v + 1]);
  L.hull[2 * v] = s1 > s0 ? L.seg[2 * (size_t)s0] : 0u;
  L.hull[2 * v + 1] = s1 > s0 ? L.seg[2 * (size_t)s1 - 1] : 0u;
}

// ---- 5c. tile live-ins ------------------------------------------------------------------
// Tile t starts at instruction t * tile_len; its seed is the set live before that
// instruction.  Replaying every occupancy event of the program from the start (nothing is
// live into the entry) gives exactly that set, and every event flips one bit, so the seed
// of tile t is the exclusive-or of all flips of the tiles before it.
// k_tile_delta: one workgroup per tile XORs the tile's flips into an LDS row: the events
// of its instructions (an occurrence with an odd number of roles flips its vreg) and of
// the block boundaries right after its instructions (live-out of the earlier block XOR
// live-in of the later one).
__device__ inline void f_tile_delta(const DevProg VL_CONSTANT &m, const DevLive VL_CONSTANT &L, const uint32_t bx, const uint32_t tx,
                                    const uint32_t bdim) {
  extern __shared__ uint32_t row[];
  const uint32_t t = bx;
  if (t >= L.T) return;
  const uint32_t W = m.W, i0 = t * L.tile_len, i1 = min(m.N, i0 + L.tile_len);
  for (uint32_t w = tx; w < W; w += 256) row[w] = 0;
  __syncthreads();
  const uint32_t o_end = m.occ_off[i1];
  for (uint32_t o = m.occ_off[i0] + tx; o < o_end; o += 4 * 256) {   // four reads of each kind in flight
    uint32_t role[4], vv[4];
#pragma unroll
    for (uint32_t u = 0; u < 4; ++u) {
      const uint32_t x = o + u * 256;
      role[u] = x < o_end ? (uint32_t)L.occ_role[x] : 0u;
      vv[u] = x < o_end ? m.occ_vreg[x] : 0u;
    }
#pragma unroll
    for (uint32_t u = 0; u < 4; ++u)
      if (__popc(role[u] & (kRolePreKill | kRoleTestSet | kRolePostKill)) & 1) atomicXor(&row[vv[u] >> 5], 1u << (vv[u] & 31));
  }
  // boundaries b whose last earlier instruction (blk_start[b] - 1) lies in this tile
  const uint32_t b_lo = m.instr_blk[i0] + 1, b_hi = m.instr_blk[i1 - 1] + 1;   // blocks starting in (i0, i1]
  for (uint32_t b = b_lo; b <= b_hi && b < m.B; ++b) {
    if (m.blk_start[b] - 1 < i0 || m.blk_start[b] - 1 >= i1) continue;
    for (uint32_t w = tx; w < W; w += 256)
      atomicXor(&row[w], L.live_out[(size_t)(b - 1) * W + w] ^ L.live_in[(size_t)b * W + w]);
  }
  __syncthreads();
  for (uint32_t w = tx; w < W; w += 256) L.tile_live[(size_t)t * W + w] = row[w];
}

// Exclusive prefix-XOR over the tiles: a lane per bitset word, and a wavefront per run of tiles where
// the words leave some of the workgroup's sixteen free (a program of 8,000 instructions has 188 words
// and 63 tiles: five runs of 13, read at once).  members: counts the members of each tile's row
// (nothing is live into the first).
constexpr uint32_t kTileWords = 1024;    // words of a workgroup
constexpr uint32_t kTileCounts = 2048;   // most tiles whose members are counted
__device__ inline void f_tile_prefix(const DevProg VL_CONSTANT &m, const DevLive VL_CONSTANT &L, const uint32_t bx, uint32_t *members) {
  __shared__ uint32_t run_xor[16][64];
  const uint32_t W = m.W, T = L.T, w0 = bx * kTileWords, lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
  if (w0 >= W) return;
  const uint32_t groups = (min(W - w0, kTileWords) + 63u) / 64u, runs = 16u / groups, run = wave / groups;
  const uint32_t w = w0 + wave % groups * 64 + lane, len = (T + runs - 1) / runs;
  const uint32_t t_lo = run < runs ? min(T, run * len) : T, t_hi = run < runs ? min(T, t_lo + len) : T;
  uint32_t d[16], x = 0;
  auto fetch = [&](uint32_t t0) __attribute__((always_inline)) {
#pragma unroll
    for (uint32_t u = 0; u < 16; ++u) d[u] = t0 + u < t_hi && w < W ? L.tile_live[(size_t)(t0 + u) * W + w] : 0u;
  };
  for (uint32_t t0 = t_lo; t0 < t_hi; t0 += 16) {
    fetch(t0);
#pragma unroll
    for (uint32_t u = 0; u < 16; ++u) x ^= d[u];
  }
  run_xor[wave][lane] = x;
  __syncthreads();
  uint32_t acc = 0;
  for (uint32_t k = wave % groups; k < run * groups && run < runs; k += groups) acc ^= run_xor[k][lane];
  for (uint32_t t0 = t_lo; t0 < t_hi; t0 += 16) {
    if (len > 16) fetch(t0);   // (otherwise they are still there)
    uint32_t two = 0;          // the counts of two tiles: a wavefront's are at most 2,048 each
#pragma unroll
    for (uint32_t u = 0; u < 16; ++u) {
      if (t0 + u < t_hi && w < W) L.tile_live[(size_t)(t0 + u) * W + w] = acc;
      if (members) {
        two |= (uint32_t)__popc(acc) << (16u * (u & 1u));
        if (u & 1u) {
          two = wave_prefix(two);
          if (lane == 63u && t0 + u - 1 < t_hi) atomicAdd(&members[t0 + u - 1], two & 0xFFFFu);
          if (lane == 63u && t0 + u < t_hi) atomicAdd(&members[t0 + u], two >> 16);
          two = 0;
        }
      }
      acc ^= d[u];
    }
  }
}

// In-place exclusive scan of p[0..n), total to p[n], by one wavefront: four elements per lane, four
// rounds of reads in flight.
__device__ inline void wave_scan(uint32_t VL_GLOBAL *p, const uint32_t n) {
  const uint32_t lane = threadIdx.x & 63u;
  uint32_t base = 0;
  for (uint32_t i0 = 0; i0 < n; i0 += 4 * 256) {
    u32x4 x[4];
#pragma unroll
    for (uint32_t u = 0; u < 4; ++u) {
      const uint32_t i = i0 + u * 256 + lane * 4;
      x[u] = 0;
#pragma unroll
      for (uint32_t t = 0; t < 4; ++t)
        if (i + t < n) x[u][t] = p[i + t];
    }
#pragma unroll
    for (uint32_t u = 0; u < 4; ++u) {
      const uint32_t i = i0 + u * 256 + lane * 4, sum = x[u].x + x[u].y + x[u].z + x[u].w, incl = wave_prefix(sum);
      uint32_t at = base + incl - sum;
#pragma unroll
      for (uint32_t t = 0; t < 4; ++t) {
        if (i + t < n) p[i + t] = at;
        at += x[u][t];
      }
      base += (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
    }
  }
  if (lane == 0) p[n] = base;
}

// One wavefront per tile lists the members of its seed row as occupy-without-test entries
// whose register is taken from the nearest earlier occurrence of the vreg.
template <bool kFill>
__device__ inline void f_seed(const DevProg VL_CONSTANT &m, const DevLive VL_CONSTANT &L, const uint32_t bx, const uint32_t tx,
                              const uint32_t bdim) {
  const uint32_t t = bx, lane = tx;
  if (t >= L.T) return;
  const uint32_t W = m.W;
  uint32_t total = 0;
  const uint32_t base = kFill ? L.seed_off[t] : 0;
  if (!kFill) {   // counting needs no positions: one reduction at the end
    uint32_t mine = 0;
    if (t > 0)
      for (uint32_t w = lane; w < W; w += 64) mine += __popc(L.tile_live[(size_t)t * W + w]);
    for (int d = 32; d >= 1; d >>= 1) mine += (uint32_t)__shfl_xor((int)mine, d, 64);
    if (lane == 0) L.seed_off[t] = mine;
    return;
  }
  for (uint32_t w0 = 0; w0 < W; w0 += 64) {
    const uint32_t w = w0 + lane;
    uint32_t bits = (w < W && t > 0) ? L.tile_live[(size_t)t * W + w] : 0u;
    const uint32_t c = __popc(bits), incl = wave_incl_scan(c);
    if (kFill) {
      uint32_t pos = base + total + incl - c;
      while (bits) {
        const uint32_t v = w * 32 + __ffs(bits) - 1;
        bits &= bits - 1;
        u32x4 r = {v, t, 0u, 0u};   // completed by k_seed_src
        L.seeds[pos++] = r;
      }
    }
    total += __shfl(incl, 63, 64);
  }
  if (!kFill && lane == 0) L.seed_off[t] = total;
}

// completes each seed entry: the register comes from the nearest earlier occurrence
__device__ inline void f_seed_src(const DevProg VL_CONSTANT &m, const DevLive VL_CONSTANT &L, const uint32_t bx, const uint32_t tx,
                                  const uint32_t bdim) {
  const uint32_t k = bx * bdim + tx;
  if (k >= L.n_seed) return;
  const u32x4 raw = L.seeds[k];
  const uint32_t v = raw.x, t = raw.y;
  // the register is always gathered from memory: the ring offset stays unused
  const uint32_t at = t * L.tile_len, lo = L.vcnt[v], hi = L.vcnt[v + 1];
  const uint32_t x = first_entry_at(L, lo, hi, at);   // first mention at or after the tile's start
  u32x4 r = event_record(m, x > lo ? L.ent[x - 1].x : (x < hi ? L.ent[x].x : 0u), v, false, true);
  r.x &= ~0xFFu;   // only the vreg: the register is always gathered from memory
  // the verifier keeps the gathered registers at hand for the link of that first mention
  if (x > lo && x < hi && (L.ent[x].y >> 2) < min(m.N, at + L.tile_len)) r.w |= kSeedLinked;
  L.seeds[k] = r;
}

// Clears `vecs` 16-byte vectors.  A kernel rather than a memset so that a caller may record
// the steady-state analysis into a stream capture (the arenas are 256-byte aligned and every
// region's length is a multiple of 256 bytes).
__global__ void k_zero(u32x4 VL_GLOBAL *p, size_t vecs) {
  const u32x4 z = {0, 0, 0, 0};
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < vecs; i += (size_t)gridDim.x * blockDim.x) p[i] = z;
}

static inline void zero_async(void *p, size_t bytes, hipStream_t stream) {
  if (!bytes) return;
  const size_t vecs = bytes / 16;
  const uint32_t blocks = (uint32_t)std::min<size_t>(8192, (vecs + 255) / 256);
  k_zero<<<blocks, 256, 0, stream>>>((u32x4 VL_GLOBAL *)p, vecs);
}

__global__ void k_collect(MIRS, uint32_t n) {
  uint32_t k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  const DevProg VL_CONSTANT &m = as_constant(mirs)[k];
  const DevLive VL_CONSTANT &L = as_constant(lives)[k];
  L.counters[kCtrPlanLen] = L.item_base[stretches(m.N)] + L.bound_off[m.B];
  L.counters[kCtrSeg] = L.seg_base[stretches(m.O)];
  L.counters[kCtrSeed] = L.seed_off[L.T];
}

__device__ inline void f_tile_range(const DevProg VL_CONSTANT &m, const DevLive VL_CONSTANT &L, const uint32_t bx, const uint32_t tx,
                                    const uint32_t bdim) {
  uint32_t t = bx * bdim + tx;
  if (t >= L.T) return;
  const uint32_t i0 = t * L.tile_len, i1 = min(m.N, i0 + L.tile_len);
  L.tile_range[2 * t] = L.item_off[item_of_instr(m, i0)];
  uint32_t end;
  if (i1 == m.N) end = L.item_off[m.N + m.B];
  else {
    const uint32_t b = m.instr_blk[i1];
    // a tile ending at a block boundary leaves the boundary entries out: the next tile
    // starts from that block's live-in
    end = m.blk_start[b] == i1 ? L.item_off[i1 + b] : L.item_off[i1 + b + 1];
  }
  L.tile_range[2 * t + 1] = end;
}

// ---- 5d. dense per-point bitsets (optional) ---------------------------------------------
// Every occupy / release event flips one bit of the occupied set.  A workgroup takes 64 bitset
// words of one tile: 64 instructions at a time, it XORs each event into the LDS row of the
// instruction at which it takes effect (an event per thread, its row found by bisection in the
// rows' first events), then prefix-XORs the rows downwards from the tile's live-in row, four
// wavefronts with 16 rows each, and writes every row once.  What changes at a block boundary comes from
// the two blocks' sets, not from the boundary's events, so that nothing here waits for those and a call of
// few programs needs no launch for it (2,000 instructions: 47.6 -> 43.6 us a call).
// (A pass of global atomics over cleared rows, an instruction per lane, and a second pass that prefixed
// them in place took 33 and 48 us for 2,000 instructions and 1,500 vregs: a lane with a block boundary's events walked them
// one by one, and the prefix waited for memory at every row.)
constexpr uint32_t kDenseRows = 64;
__device__ inline void f_dense(const DevProg VL_CONSTANT &m, const DevLive VL_CONSTANT &L, const uint32_t t, const uint32_t w0) {
  const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6, w = w0 + lane;
  if (t >= L.T || w0 >= m.W) return;
  // per row: its events [start, stop), and the block that begins there (0: none, or the tile does too)
  __shared__ uint32_t rows[kDenseRows][64], start[kDenseRows], stop[kDenseRows], begins[kDenseRows], total[4][64];
  constexpr uint32_t kPer = kDenseRows / 4;
  const uint32_t i0 = t * L.tile_len, i1 = min(m.N, i0 + L.tile_len);
  uint32_t cur = t && w < m.W ? L.tile_live[(size_t)t * m.W + w] : 0u;
  for (uint32_t c0 = i0; c0 < i1; c0 += kDenseRows) {
    const uint32_t n = min(kDenseRows, i1 - c0);
    if (threadIdx.x < kDenseRows) {
      const uint32_t i = min(c0 + threadIdx.x, i1 - 1), b = m.instr_blk[i], item = i + b + 1;
      start[threadIdx.x] = L.item_off[item];
      stop[threadIdx.x] = L.item_off[item + 1];
      begins[threadIdx.x] = threadIdx.x < n && i != i0 && m.blk_start[b] == i ? b : 0u;
    }
#pragma unroll
    for (uint32_t k = 0; k < kPer; ++k) rows[wave * kPer + k][lane] = 0;
    __syncthreads();
    for (uint32_t e = start[0] + threadIdx.x; e < stop[n - 1]; e += 256) {
      uint32_t lo = 0, hi = n;   // the last row whose first event is e or earlier
      while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (start[mid] <= e) lo = mid; else hi = mid;
      }
      if (e >= stop[lo]) continue;   // a boundary's
      const uint32_t v = L.plan[e].x >> 8, col = (v >> 5) - w0;
      if (col < 64) atomicXor(&rows[lo][col], 1u << (v & 31));
    }
    __syncthreads();
    uint32_t x = 0, down[kPer];
#pragma unroll
    for (uint32_t k = 0; k < kPer; ++k) {
      const uint32_t b = __builtin_amdgcn_readfirstlane(begins[wave * kPer + k]);
      if (b && w < m.W) x ^= L.live_out[(size_t)(b - 1) * m.W + w] ^ L.live_in[(size_t)b * m.W + w];
      down[k] = x ^= rows[wave * kPer + k][lane];
    }
    total[wave][lane] = x;
    __syncthreads();
    uint32_t above = cur;
#pragma unroll
    for (uint32_t k = 0; k < 4; ++k) {
      above ^= k < wave ? total[k][lane] : 0u;
      cur ^= total[k][lane];
    }
#pragma unroll
    for (uint32_t k = 0; k < kPer; ++k) {
      const uint32_t r = wave * kPer + k;
      if (r < n && w < m.W) L.live_after[(size_t)(c0 + r) * m.W + w] = above ^ down[k];
    }
    __syncthreads();   // the shared rows are cleared for the next ones
  }
}

__global__ __launch_bounds__(256) void k_dense(MIRS) {
  f_dense(as_constant(mirs)[blockIdx.z], as_constant(lives)[blockIdx.z], blockIdx.y, blockIdx.x * 64);
}

// ---- stages ---------------------------------------------------------------------------
// After the per-occurrence pass three chains are independent: the event stream (counts, prefix,
// fill, chunk cuts), the intervals (counts, prefix, fill, offsets) and the tile live-ins (flips,
// prefix, counts, fill, sources).  Each stage below runs one step of every chain in one launch, the
// block index selecting the part, so that the short serial steps of one chain (prefixes) overlap the
// bandwidth-heavy steps of another.  A part made of one wavefront per item gets four items per
// 256-thread block.  Counts are prefixed per stretch of 256 where they are counted, so that only the
// stretches' totals have to be scanned in between, and a stretch's first place is a look-up for the
// kernels that fill.  (Scanning every entry and every instruction, and offsets, counts of the
// live-ins and their scan in two launches of their own: 38 us for 256 programs of 1,000-20,000
// instructions and 22 for one of 8,000, where the one launch takes 11.5 and 7.5.)
struct StageGrid { uint32_t a, b, c; };   // blocks of the three parts, in launch order

__global__ __launch_bounds__(256) void k_stage_count(MIRS, const Grid grid, StageGrid g) {
  const uint32_t prog = grid_prog(grid), bx = grid_block(grid);
  if (prog >= grid.n) return;
  const DevProg VL_CONSTANT &m = as_constant(mirs)[prog];
  const DevLive VL_CONSTANT &L = as_constant(lives)[prog];
  const uint32_t tx = threadIdx.x;
  if (bx < g.a) f_tile_delta(m, L, bx, tx, 256);
  else if (bx < g.a + g.b) f_boundary<false>(m, L, (bx - g.a) * 4 + (tx >> 6), tx & 63u, 64);
  else f_item_count(m, L, bx - g.a - g.b, tx);
}

// kCount: a workgroup per kernel does everything, its wavefronts side by side; otherwise the tiles'
// rows are prefixed by workgroups of their own.
constexpr uint32_t kWaveScan = 4096;   // longer arrays are scanned by the whole workgroup
template <bool kCount>
__global__ __launch_bounds__(1024) void k_stage_scan(MIRS) {
  const DevProg VL_CONSTANT &m = as_constant(mirs)[blockIdx.y];
  const DevLive VL_CONSTANT &L = as_constant(lives)[blockIdx.y];
  if (!kCount && blockIdx.x > 0) {
    f_tile_prefix(m, L, blockIdx.x - 1, nullptr);
    return;
  }
  __shared__ uint32_t members[kCount ? kTileCounts : 1];
  if (kCount) {
    for (uint32_t t = threadIdx.x; t < L.T; t += 1024) members[t] = 0;
    __syncthreads();
    f_tile_prefix(m, L, 0, members);
    __syncthreads();
  }
  const uint32_t wave = threadIdx.x >> 6, lane = threadIdx.x & 63u;
  if (kCount && wave == 3) {
    uint32_t base = 0;
    for (uint32_t t0 = 0; t0 < L.T; t0 += 64) {
      const uint32_t t = t0 + lane, x = t < L.T ? members[t] : 0u, incl = wave_prefix(x);
      if (t < L.T) L.seed_off[t] = base + incl - x;
      base += (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
    }
    if (lane == 0) L.seed_off[L.T] = base;
  }
  if (max(max(m.O, m.N) / kStretch, m.B) < kWaveScan) {
    if (wave == 0) wave_scan(L.seg_base, stretches(m.O));
    if (wave == 1) wave_scan(L.item_base, stretches(m.N));
    if (wave == 2) wave_scan(L.bound_off, m.B);
  } else {
    f_scan<kScanSeg>(m, L);
    __syncthreads();
    f_scan<kScanItems>(m, L);
    __syncthreads();
    f_scan<kScanBound>(m, L);
  }
}

// the counts of the tiles' live-ins where a row takes several workgroups of the launch above
__global__ __launch_bounds__(256) void k_seed_count(MIRS) {
  f_seed<false>(as_constant(mirs)[blockIdx.y], as_constant(lives)[blockIdx.y], blockIdx.x * 4 + (threadIdx.x >> 6), threadIdx.x & 63u, 64);
}

// One-dimensional grid.  Part a: per_a workgroups for every kernel; parts b and c: one
// workgroup per stretch of 256 instructions / entries that exists, named by the block maps.
// (Where programs are dealt out to the dies, each part begins at a multiple of eight.)
__global__ __launch_bounds__(256) void k_stage_fill(MIRS, const Grid grid, StageGrid g, uint32_t per_a, const uint2 *__restrict__ map_instr,
                                                    const uint2 *__restrict__ map_occ) {
  const uint32_t bx = blockIdx.x, tx = threadIdx.x;
  uint2 where;
  if (bx < g.a) {
    const uint32_t per_row = per_a << grid.dealt, y = bx / per_row, x = bx - y * per_row;
    where = make_uint2((y << grid.dealt) + (x & ((1u << grid.dealt) - 1u)), x >> grid.dealt);
  }
  else if (bx < g.a + g.b) where = map_instr ? map_instr[bx - g.a] : make_uint2(0, bx - g.a);
  else where = map_occ ? map_occ[bx - g.a - g.b] : make_uint2(0, bx - g.a - g.b);
  if (where.x >= grid.n) return;
  const DevProg VL_CONSTANT &m = as_constant(mirs)[where.x];
  const DevLive VL_CONSTANT &L = as_constant(lives)[where.x];
  if (bx < g.a) f_seed<true>(m, L, where.y * 4 + (tx >> 6), tx & 63u, 64);
  else if (bx < g.a + g.b) f_plan_fill(m, L, where.y, tx, 256);
  else f_seg_fill(m, L, where.y, tx, 256);
}

// kDense: the first n_dense workgroups of a program write its dense points, across words 64 at a time, then tiles
template <bool kDense>
__global__ __launch_bounds__(256) void k_stage_finish(MIRS, const Grid grid, StageGrid g, uint32_t n_dense, uint32_t across) {
  const uint32_t prog = grid_prog(grid);
  uint32_t bx = grid_block(grid);
  if (prog >= grid.n) return;
  const DevProg VL_CONSTANT &m = as_constant(mirs)[prog];
  const DevLive VL_CONSTANT &L = as_constant(lives)[prog];
  const uint32_t tx = threadIdx.x;
  if (kDense) {
    if (bx < n_dense) {
      f_dense(m, L, bx / across, bx % across * 64);
      return;
    }
    bx -= n_dense;
  }
  if (bx < g.a) f_boundary<true>(m, L, bx * 4 + (tx >> 6), tx & 63u, 64);
  else if (bx < g.a + g.b) f_tile_range(m, L, bx - g.a, tx, 256);
  else if (bx < g.a + g.b + g.c) f_seed_src(m, L, bx - g.a - g.b, tx, 256);
  else f_hull(m, L, bx - g.a - g.b - g.c, tx, 256);
}

struct Bump {
  size_t off = 0;
  size_t take(size_t bytes) {
    size_t at = off;
    off += (bytes + 255) & ~(size_t)255;
    return at;
  }
};

}  // namespace

// A batch owns the device storage of n analyses made by one call.
struct vl_batch {
  uint32_t n = 0, refs = 0;
  int device = 0;
  void *arena1 = nullptr, *arena2 = nullptr;
  size_t cap1 = 0, cap2 = 0;
  DevProg *dev_mirs = nullptr;        // device array [n]
  DevLive *dev_lives = nullptr;       // device array [n]
  void *pinned = nullptr;             // one allocation that holds the five arrays below
  uint32_t *host_counters = nullptr;  // [n][kCounters]
  DevProg *stage_mirs = nullptr;      // [n]
  DevLive *stage_a = nullptr, *stage_b = nullptr;  // [n] each: first and second upload
  uint2 *stage_map = nullptr;         // the block maps (kernel, stretch of 256) of the per-instruction and per-entry launches
  // The order of the batch's programs in the device tables, and the sizes of the block maps.  dealt:
  // program k stays on die place[k] % 8 (see Grid).
  std::vector<uint32_t> place;   // [n]
  bool dealt = false;
  size_t blocks_instr = 0, blocks_occ = 0;
  std::vector<vl_live *> lives;
  // result sizes of the last successful call (the analysis of the same kernels with the same
  // options is deterministic, so a recycling call need not read them back)
  bool sized = false, sized_dense = false;
  uint32_t sized_tile_len = 0;
  std::vector<uint32_t> sizes;   // [n][3]: events, interval segments, tile live-ins
  std::vector<char> uploaded;    // the DevLive table as it stands on the device after the last successful call
};

// Device memory of analyses on its way from one to the next.  Kernels that arrive with their first
// samples are analysed into new handles and dropped, and mapping and unmapping tens of megabytes
// took longer than the analysis (32 MB: hipMalloc 24 us, hipFree 180 us).  A few blocks of middling
// size per device are kept when an analysis is destroyed; a block that several takers in turn had no
// use for goes back to the system, and all of them when any allocation of the library finds memory short.  As with hipFree, whoever
// gives memory back waits for the device, so what a taker gets is idle on every stream.
namespace {
struct Arena {
  void *mem;
  size_t cap;
};
constexpr int kPoolBlocks = 6;
constexpr size_t kPoolMin = 1u << 20, kPoolMax = 64u << 20;   // bytes of a block that is kept
constexpr uint32_t kPoolIdle = 32;                            // takers that pass a block by before it is freed
struct Pool {
  std::mutex mu;
  Arena block[kPoolBlocks] = {};
  uint32_t passed[kPoolBlocks] = {};
};
Pool g_pool[16];

// gives back everything that is kept; whether that was anything
bool pool_empty(int device) {
  if (device < 0 || device >= 16) return false;
  Arena all[kPoolBlocks];
  {
    std::lock_guard<std::mutex> lock(g_pool[device].mu);
    for (int k = 0; k < kPoolBlocks; ++k) { all[k] = g_pool[device].block[k]; g_pool[device].block[k] = {nullptr, 0}; }
  }
  bool any = false;
  for (const Arena &a : all)
    if (a.mem) { (void)hipFree(a.mem); any = true; }
  return any;
}
}  // namespace

hipError_t vl::device_alloc(void **mem, size_t bytes) {
  hipError_t e = hipMalloc(mem, bytes);
  if (e != hipErrorOutOfMemory) return e;
  (void)hipGetLastError();
  int device = 0;
  if (hipGetDevice(&device) != hipSuccess || !pool_empty(device)) return e;
  return hipMalloc(mem, bytes);
}

namespace {
hipError_t arena_take(int device, size_t bytes, void **mem, size_t *cap) {
  Arena got = {nullptr, 0}, stale[kPoolBlocks] = {};
  Pool *pool = device >= 0 && device < 16 ? &g_pool[device] : nullptr;
  if (pool) {
    std::lock_guard<std::mutex> lock(pool->mu);
    int best = -1;
    for (int k = 0; k < kPoolBlocks; ++k)
      if (pool->block[k].mem && pool->block[k].cap >= bytes && pool->block[k].cap / 4 <= bytes && (best < 0 || pool->block[k].cap < pool->block[best].cap)) best = k;
    for (int k = 0; k < kPoolBlocks; ++k) {
      if (k == best) got = pool->block[k];
      else if (pool->block[k].mem && ++pool->passed[k] > kPoolIdle) stale[k] = pool->block[k];
      else continue;
      pool->block[k] = {nullptr, 0};
    }
  }
  for (const Arena &a : stale)
    if (a.mem) (void)hipFree(a.mem);
  hipError_t e = hipSuccess;
  if (!got.mem) {
    got.cap = bytes;
    e = device_alloc(&got.mem, bytes);
    if (e != hipSuccess) got = {nullptr, 0};
  }
  *mem = got.mem;
  *cap = got.cap;
  return e;
}

void arenas_give(int device, std::initializer_list<Arena> arenas) {
  bool worth = false;
  for (const Arena &a : arenas) worth |= a.mem && a.cap >= kPoolMin && a.cap <= kPoolMax;
  Pool *pool = device >= 0 && device < 16 && worth ? &g_pool[device] : nullptr;
  if (pool) {
    int before = device;
    bool idle = hipGetDevice(&before) == hipSuccess && (before == device || hipSetDevice(device) == hipSuccess);
    idle = idle && hipDeviceSynchronize() == hipSuccess;
    if (before != device) (void)hipSetDevice(before);
    if (!idle) pool = nullptr;   // (hipFree below waits, or says what is wrong)
  }
  for (const Arena &a : arenas) {
    if (!a.mem) continue;
    bool kept = false;
    if (pool && a.cap >= kPoolMin && a.cap <= kPoolMax) {
      std::lock_guard<std::mutex> lock(pool->mu);
      for (int k = 0; k < kPoolBlocks && !kept; ++k)
        if (!pool->block[k].mem) {
          pool->block[k] = a;
          pool->passed[k] = 0;
          kept = true;
        }
    }
    if (!kept) (void)hipFree(a.mem);
  }
}
}  // namespace

static void batch_free(vl_batch *b) {
  arenas_give(b->device, {{b->arena1, b->cap1}, {b->arena2, b->cap2}});
  if (b->pinned) (void)hipHostFree(b->pinned);
  delete b;
}

extern "C" void vl_live_destroy(vl_live *l) {
  if (!l || l->magic != kLiveMagic) return;
  l->magic = 0;
  vl_batch *b = l->batch;
  delete l;
  if (--b->refs == 0) batch_free(b);
}

// Deals the programs out to the eight dies where that leaves the dies equally busy: by size, to and fro.
// A batch of few or very unequal programs, one of whose dies would get a sixteenth more than the
// mean, stays in the caller's order, every program spread over all dies; so does one so large that the
// empty blocks which fill up a die could make a launch larger than a grid can be (2^24 blocks of 256).
constexpr uint64_t kDealtBlocks = 1u << 22;
static void deal(vl_batch *batch, const vl_mir *const *mirs) {
  const uint32_t n = batch->n;
  std::vector<uint32_t> by_size(n);
  for (uint32_t k = 0; k < n; ++k) by_size[k] = k;
  batch->place = by_size;
  uint64_t instr[8] = {}, occ[8] = {}, sum_instr = 0, sum_occ = 0, max_instr = 0, max_occ = 0;
  std::stable_sort(by_size.begin(), by_size.end(), [&](uint32_t a, uint32_t b) { return mirs[a]->h.O > mirs[b]->h.O; });
  auto place_of = [&](uint32_t r) { return (r & 8u) && (r | 7u) < n ? r ^ 7u : r; };   // every second row of eight backwards
  for (uint32_t r = 0; r < n; ++r) {
    const DevMir &m = mirs[by_size[r]]->h;
    instr[place_of(r) % 8] += stretches(m.N);
    occ[place_of(r) % 8] += stretches(m.O);
  }
  for (uint32_t d = 0; d < 8; ++d) {
    sum_instr += instr[d];
    sum_occ += occ[d];
    max_instr = std::max(max_instr, instr[d]);
    max_occ = std::max(max_occ, occ[d]);
  }
  batch->dealt = n >= 8 && 8 * max_occ <= sum_occ + sum_occ / 16 && 8 * max_instr <= sum_instr + sum_instr / 16 && 8 * (max_instr + max_occ) <= kDealtBlocks;
  if (batch->dealt)
    for (uint32_t r = 0; r < n; ++r) batch->place[by_size[r]] = place_of(r);
  batch->blocks_instr = batch->dealt ? 8 * max_instr : sum_instr;
  batch->blocks_occ = batch->dealt ? 8 * max_occ : sum_occ;
}

extern "C" int32_t vl_liveness_multi(const vl_mir *const *mirs, uint32_t n, uint32_t flags, uint32_t tile_len,
                                     vl_stream stream_, vl_live **live) {
  if (!mirs || !live) return VL_E_NULL;
  if (n == 0 || n > 65535) return VL_E_SHAPE;
  if (flags & ~VL_DENSE_POINTS) return VL_E_RANGE;
  for (uint32_t k = 0; k < n; ++k)
    if (!mirs[k] || mirs[k]->magic != kMirMagic) return VL_E_NULL;
  hipStream_t stream = (hipStream_t)stream_;
  uint32_t span = 1;   // tiles a verification may join: up to 128 instructions, where the length is not the caller's
  if (tile_len == 0) {
    // Default: 512 instructions per tile when that gives the verifier a thousand tiles or more
    // over the batch; a small batch gets shorter tiles (down to 128), so that its candidate
    // walk has workgroups for more of the device (one kernel of 8,000 instructions with 1,000
    // candidates: 0.043 ms with tiles of 128 against 0.091 ms with tiles of 512).
    uint64_t total = 0;
    for (uint32_t k = 0; k < n; ++k) total += mirs[k]->h.N;
    tile_len = kDefaultTile;
    while (tile_len > 128 && total / tile_len < 1024) tile_len /= 2;
    // What makes fewer than 48 of those leaves most of the device without work, and is cut down to 32
    // (200 instructions with 64 samples: 24.9 us a call with tiles of 128, 18.3 with 32; 4,000 with 100
    // samples: 51, and 40 with 64).  Where there are enough samples to fill the device with longer tiles, a
    // verification joins them again, up to 128 instructions.
    while (tile_len > 32 && total / tile_len < 48) { tile_len /= 2; span *= 2; }
  }
  const bool dense = (flags & VL_DENSE_POINTS) != 0;

  // recycle or create the batch
  vl_batch *batch = nullptr;
  bool fresh = false;
  if (live[0]) {
    for (uint32_t k = 0; k < n; ++k) {
      if (!live[k] || live[k]->magic != kLiveMagic || live[k]->index != k) return VL_E_ARG;
      if (live[k]->batch != live[0]->batch || live[k]->mir != mirs[k]) return VL_E_ARG;
    }
    batch = live[0]->batch;
    if (batch->n != n) return VL_E_ARG;
  } else {
    for (uint32_t k = 0; k < n; ++k)
      if (live[k]) return VL_E_ARG;
    batch = new (std::nothrow) vl_batch;
    if (!batch) return VL_E_SHAPE;
    batch->n = n;
    fresh = true;
    deal(batch, mirs);
    // block maps: one entry per stretch of 256 instructions, then one per stretch of 256 entries
    const size_t blocks_instr = batch->blocks_instr, blocks_occ = batch->blocks_occ;
    const bool too_many = blocks_instr + blocks_occ > 0x7FFFFFFFull;
    if (too_many) { delete batch; return VL_E_RANGE; }
    hipError_t e = hipGetDevice(&batch->device);
    Bump pin;
    const size_t o_cnt = pin.take((size_t)n * kCounters * 4), o_mir = pin.take((size_t)n * sizeof(DevProg));
    const size_t o_a = pin.take((size_t)n * sizeof(DevLive)), o_b = pin.take((size_t)n * sizeof(DevLive));
    const size_t o_map = pin.take((blocks_instr + blocks_occ + 1) * sizeof(uint2));
    if (e == hipSuccess) e = hipHostMalloc(&batch->pinned, pin.off, hipHostMallocDefault);
    if (e == hipSuccess) {
      char *at = (char *)batch->pinned;
      batch->host_counters = (uint32_t *)(at + o_cnt);
      batch->stage_mirs = (DevProg *)(at + o_mir);
      batch->stage_a = (DevLive *)(at + o_a); batch->stage_b = (DevLive *)(at + o_b);
      batch->stage_map = (uint2 *)(at + o_map);
    }
    if (e != hipSuccess) { batch_free(batch); return hip_fail(e); }
  }
  auto fail = [&](int32_t rc) {
    if (fresh) batch_free(batch);
    return rc;
  };

  const size_t blocks_instr = batch->blocks_instr, blocks_occ = batch->blocks_occ;
  const std::vector<uint32_t> &place = batch->place;
  // the tables in the order they have on the device
  auto placed = [&](const std::vector<DevLive> &from, DevLive *to) {
    for (uint32_t k = 0; k < n; ++k) to[place[k]] = from[k];
  };

  // ---- arena 1 layout: [zeroed zone | counters | rest | device tables] ----
  std::vector<DevLive> h(n);
  struct Off1 { size_t last_live, vcnt, vcur, use, def, in, seed_off, out, tmp, vocc, ent, ent_info, first, prev,
                role, kill, item, seg_off, hull, queue, ent_seg, ent_sf, chk, evt_cut, tile_live, seg_base, item_base, bound_off; };
  std::vector<Off1> off(n);
  Bump bump;
  uint32_t maxO = 1, maxV = 1, maxN = 1, maxB = 1, maxW = 1, maxT = 1, maxE = 0;
  for (uint32_t k = 0; k < n; ++k) {
    const DevMir &m = mirs[k]->h;
    const uint32_t T = (m.N + tile_len - 1) / tile_len;
    memset(&h[k], 0, sizeof(DevLive));
    h[k].T = T; h[k].tile_len = tile_len; h[k].dense = dense;
    const size_t bw = (size_t)m.B * std::max(1u, m.W) * 4;
    off[k].vcnt = bump.take((size_t)(m.V + 1) * 4);
    off[k].vcur = bump.take((size_t)(m.V + 1) * 4);
    off[k].last_live = bump.take((size_t)(m.V + 1) * 4);
    off[k].use = bump.take(bw); off[k].def = bump.take(bw); off[k].in = bump.take(bw);
    off[k].seed_off = bump.take((size_t)(T + 1) * 4);
    off[k].item = bump.take((size_t)(m.N + m.B + 1) * 4);
    maxO = std::max(maxO, m.O); maxV = std::max(maxV, m.V); maxN = std::max(maxN, m.N);
    maxB = std::max(maxB, m.B); maxW = std::max(maxW, m.W); maxT = std::max(maxT, T); maxE = std::max(maxE, m.E);
  }
  const size_t o_counters = bump.take((size_t)n * kCounters * 4);
  const size_t zero_bytes = bump.off;
  for (uint32_t k = 0; k < n; ++k) {
    const DevMir &m = mirs[k]->h;
    const size_t O1 = std::max(1u, m.O), bw = (size_t)m.B * std::max(1u, m.W) * 4;
    off[k].out = bump.take(bw);
    off[k].tmp = bump.take(O1 * 4); off[k].vocc = bump.take(O1 * 4); off[k].ent = bump.take(O1 * sizeof(u32x4));
    off[k].ent_info = bump.take(O1); off[k].first = bump.take((size_t)(m.V + 1) * 4); off[k].prev = bump.take(O1 * 4);
    off[k].role = bump.take(O1); off[k].kill = bump.take(O1);
    off[k].seg_off = bump.take((size_t)(m.V + 1) * 4); off[k].hull = bump.take((size_t)(m.V + 1) * 8);
    off[k].queue = bump.take((size_t)(m.V + 1) * 4);
    off[k].ent_seg = bump.take((O1 + 1) * 4);
    off[k].ent_sf = bump.take(O1);
    off[k].chk = bump.take(O1 * sizeof(u32x4));
    off[k].tile_live = bump.take((size_t)h[k].T * std::max(1u, m.W) * 4);
    off[k].evt_cut = bump.take(((size_t)(m.O + 63) / 64 + 2) * 4);
    off[k].seg_base = bump.take(((size_t)stretches(m.O) + 1) * 4);
    off[k].item_base = bump.take(((size_t)stretches(m.N) + 1) * 4);
    off[k].bound_off = bump.take(((size_t)m.B + 1) * 4);
  }
  const size_t o_mirs = bump.take((size_t)n * sizeof(DevProg));
  const size_t o_lives = bump.take((size_t)n * sizeof(DevLive));
  const size_t o_map = bump.take((blocks_instr + blocks_occ + 1) * sizeof(uint2));
  if (bump.off > batch->cap1) {
    if (batch->arena1) { VL_HIP(hipStreamSynchronize(stream)); (void)hipFree(batch->arena1); batch->arena1 = nullptr; batch->cap1 = 0; }
    hipError_t e = arena_take(batch->device, bump.off, &batch->arena1, &batch->cap1);
    if (e != hipSuccess) return fail(hip_fail(e));
  }
  char *a1 = (char *)batch->arena1;
  DevProg *const progs = batch->stage_mirs;
  for (uint32_t k = 0; k < n; ++k) {
    DevLive &L = h[k];
    L.vcnt = (uint32_t VL_GLOBAL *)(a1 + off[k].vcnt); L.vcur = (uint32_t VL_GLOBAL *)(a1 + off[k].vcur);
    L.last_live = (uint32_t VL_GLOBAL *)(a1 + off[k].last_live);
    L.use = (uint32_t VL_GLOBAL *)(a1 + off[k].use); L.def = (uint32_t VL_GLOBAL *)(a1 + off[k].def);
    L.live_in = (uint32_t VL_GLOBAL *)(a1 + off[k].in); L.live_out = (uint32_t VL_GLOBAL *)(a1 + off[k].out);
    L.seed_off = (uint32_t VL_GLOBAL *)(a1 + off[k].seed_off);
    L.vocc_tmp = (uint32_t VL_GLOBAL *)(a1 + off[k].tmp); L.vocc = (uint32_t VL_GLOBAL *)(a1 + off[k].vocc);
    L.ent = (u32x4 VL_GLOBAL *)(a1 + off[k].ent); L.ent_info = (uint8_t VL_GLOBAL *)(a1 + off[k].ent_info);
    L.first = (uint32_t VL_GLOBAL *)(a1 + off[k].first); L.prev_occ = (uint32_t VL_GLOBAL *)(a1 + off[k].prev);
    L.occ_role = (uint8_t VL_GLOBAL *)(a1 + off[k].role); L.occ_kill = (uint8_t VL_GLOBAL *)(a1 + off[k].kill);
    L.item_off = (uint32_t VL_GLOBAL *)(a1 + off[k].item); L.seg_off = (uint32_t VL_GLOBAL *)(a1 + off[k].seg_off);
    L.hull = (uint32_t VL_GLOBAL *)(a1 + off[k].hull); L.long_queue = (uint32_t VL_GLOBAL *)(a1 + off[k].queue);
    L.ent_seg = (uint32_t VL_GLOBAL *)(a1 + off[k].ent_seg);
    L.ent_sf = (uint8_t VL_GLOBAL *)(a1 + off[k].ent_sf);
    L.chk = (u32x4 VL_GLOBAL *)(a1 + off[k].chk); L.tile_live = (uint32_t VL_GLOBAL *)(a1 + off[k].tile_live); L.evt_cut = (uint32_t VL_GLOBAL *)(a1 + off[k].evt_cut);
    L.seg_base = (uint32_t VL_GLOBAL *)(a1 + off[k].seg_base); L.item_base = (uint32_t VL_GLOBAL *)(a1 + off[k].item_base);
    L.bound_off = (uint32_t VL_GLOBAL *)(a1 + off[k].bound_off);
    L.counters = (uint32_t VL_GLOBAL *)(a1 + o_counters) + (size_t)k * kCounters;
    progs[place[k]] = mirs[k]->h;
  }
  batch->dev_mirs = (DevProg *)(a1 + o_mirs);
  batch->dev_lives = (DevLive *)(a1 + o_lives);
  // Recycled handles of a call with the same options: the result sizes and the absence of
  // contract violations are known from it (the analysis of the same kernels is
  // deterministic), so nothing is read back and the host does not wait.  (The pinned staging
  // buffers are then rewritten with the bytes they already hold.)  Putting the three chains
  // that are independent after the per-occurrence pass on streams of their own shortened the
  // analysis by a sixth but cost more than that in host-side event calls; it is one stream.
  const bool known = !fresh && batch->sized && batch->sized_tile_len == tile_len && batch->sized_dense == dense;
  if (!known) batch->sized = false;

  // ---- arena 2, sized from the counts ----
  struct Off2 { size_t plan, seeds, seg, range, dense; };
  std::vector<Off2> off2(n);
  uint32_t max_seed = 0;
  auto layout2 = [&]() -> int32_t {
    Bump b2;
    if (dense) {
      for (uint32_t k = 0; k < n; ++k) {
        const DevMir &m = mirs[k]->h;
        off2[k].dense = b2.take((size_t)m.N * std::max(1u, m.W) * 4);
      }
    }
    for (uint32_t k = 0; k < n; ++k) {
      h[k].plan_len = batch->sizes[3 * k]; h[k].n_seg = batch->sizes[3 * k + 1]; h[k].n_seed = batch->sizes[3 * k + 2];
      max_seed = std::max(max_seed, h[k].n_seed);
      off2[k].plan = b2.take(((size_t)h[k].plan_len + 8) * sizeof(u32x4));
      off2[k].seeds = b2.take((size_t)std::max(1u, h[k].n_seed) * sizeof(u32x4));
      off2[k].seg = b2.take((size_t)std::max(1u, h[k].n_seg) * 8);
      off2[k].range = b2.take((size_t)h[k].T * 8);
    }
    if (b2.off > batch->cap2) {
      if (batch->arena2) { (void)hipFree(batch->arena2); batch->arena2 = nullptr; batch->cap2 = 0; }
      hipError_t ae = arena_take(batch->device, b2.off, &batch->arena2, &batch->cap2);
      if (ae != hipSuccess) return hip_fail(ae);
    }
    char *a2 = (char *)batch->arena2;
    for (uint32_t k = 0; k < n; ++k) {
      DevLive &L = h[k];
      L.plan = (u32x4 VL_GLOBAL *)(a2 + off2[k].plan); L.seeds = (u32x4 VL_GLOBAL *)(a2 + off2[k].seeds);
      L.seg = (uint32_t VL_GLOBAL *)(a2 + off2[k].seg); L.tile_range = (uint32_t VL_GLOBAL *)(a2 + off2[k].range);
      L.live_after = dense ? (uint32_t VL_GLOBAL *)(a2 + off2[k].dense) : (uint32_t VL_GLOBAL *)nullptr;
    }
    return VL_OK;
  };
  if (known) {
    const int32_t rc2 = layout2();
    if (rc2 != VL_OK) return fail(rc2);
  }

  // pinned staging: stage_a / stage_mirs are read by the copies below; when the sizes are not
  // known yet the host waits further down and stage_b carries the second upload after that
  hipError_t e = hipSuccess;
  // with known sizes the tables on the device are usually the ones this call would upload
  const bool tables_current = known && batch->uploaded.size() == (size_t)n * sizeof(DevLive) &&
                              memcmp(batch->uploaded.data(), h.data(), batch->uploaded.size()) == 0;
  if (!tables_current) {
    batch->uploaded.clear();
    placed(h, batch->stage_a);
    if (e == hipSuccess) e = hipMemcpyAsync(a1 + o_mirs, progs, (size_t)n * sizeof(DevProg), hipMemcpyHostToDevice, stream);
    if (e == hipSuccess) e = hipMemcpyAsync(a1 + o_lives, batch->stage_a, (size_t)n * sizeof(DevLive), hipMemcpyHostToDevice, stream);
    if (e == hipSuccess && n > 1) {
      uint2 *const at = batch->stage_map;
      std::vector<uint32_t> prog(n);
      for (uint32_t k = 0; k < n; ++k) prog[place[k]] = k;
      // die d's blocks are the entries d, d + 8, ...; `step` 1: all in a row
      auto map_of = [&](uint2 *map, size_t len, bool occ) {
        const uint32_t step = batch->dealt ? 8u : 1u;
        for (uint32_t d = 0; d < step; ++d) {
          size_t x = d;
          for (uint32_t p = d; p < n; p += step) {
            const uint32_t all = stretches(occ ? mirs[prog[p]]->h.O : mirs[prog[p]]->h.N);
            for (uint32_t y = 0; y < all; ++y, x += step) map[x] = make_uint2(p, y);
          }
          for (; x < len; x += step) map[x] = make_uint2(kNone, 0);
        }
      };
      map_of(at, blocks_instr, false);
      map_of(at + blocks_instr, blocks_occ, true);
      e = hipMemcpyAsync(a1 + o_map, batch->stage_map, (blocks_instr + blocks_occ) * sizeof(uint2), hipMemcpyHostToDevice, stream);
    }
  }
  if (e != hipSuccess) return fail(hip_fail(e));
  // (one program's blocks are its stretches in order: no map, a trip to memory less)
  const uint2 *map_instr = n > 1 ? (const uint2 *)(a1 + o_map) : nullptr, *map_occ = n > 1 ? map_instr + blocks_instr : nullptr;

  const DevProg *dm = batch->dev_mirs;
  const DevLive *dl = batch->dev_lives;
  const uint32_t TB = 256;
  // LDS histograms over the vregs when they fit
  static const bool lds_ok = [] {
    bool ok = true;
    for (const void *f : {(const void *)k_group<true>, (const void *)k_group<false>, (const void *)k_count<true>, (const void *)k_place<true>})
      ok = ok && hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, 128 * 1024) == hipSuccess;
    return ok;
  }();
  const bool hist_lds = lds_ok && (size_t)maxV * 4 <= 128 * 1024;
  auto blocks = [](uint32_t items, uint32_t per) { return std::max(1u, (items + per - 1) / per); };
  // a launch of so many blocks for every program
  struct Launch { dim3 dim; Grid grid; };
  auto all_progs = [&](uint32_t per) {
    // (threads in a row of the grid stay below 2^32)
    return batch->dealt && per < (1u << 18) ? Launch{dim3(8 * per, (n + 7) / 8), {n, 3}} : Launch{dim3(per, n), {n, 0}};
  };
  // (k_group clears block sets by 32-bit indices)
  const bool small = hist_lds && maxO <= kGroupMaxOcc && (uint64_t)maxB * maxW < (1ull << 32) - 4;
  if (small) {
    uint32_t rounds = kGroupRounds;
    while (rounds > 2 && blocks_occ * kStretch / (rounds / 2 * kRound) + n <= kGroupFew && maxO / (rounds / 2 * kRound) < kGroupSlices) rounds /= 2;
    const Launch l = all_progs(blocks(maxO, rounds * kRound));
    static_assert(kGroupSlices * (kGroupRounds / 2) * kRound <= 1u << 16, "more slices than usual: counts of 16 bits");
    (rounds < kGroupRounds ? k_group<true> : k_group<false>)<<<l.dim, 1024, (size_t)maxV * 4, stream>>>(dm, dl, l.grid, rounds * kRound);
  } else {
    zero_async(a1, zero_bytes, stream);
    const dim3 slices((maxO + kSlice - 1) / kSlice, n);
    if (hist_lds) k_count<true><<<slices, 1024, (size_t)maxV * 4, stream>>>(dm, dl);
    else k_count<false><<<slices, 1024, 2 * kPlaces * 4, stream>>>(dm, dl);
    k_scan<kScanVreg><<<n, 1024, 0, stream>>>(dm, dl);
    if (hist_lds) k_place<true><<<slices, 1024, (size_t)maxV * 4, stream>>>(dm, dl);
    else k_place<false><<<slices, 1024, 2 * kPlaces * 4, stream>>>(dm, dl);
    k_sort<<<dim3(kLongBlocks + (maxV + 255) / 256, n), 256, 0, stream>>>(dm, dl);
  }
  {
    const size_t lds = std::min<size_t>((size_t)maxB * std::min(maxW, kOrdWords) * 8, 40 * 1024);
    const Launch l = all_progs(blocks(maxO, kOrdStretch));
    const uint32_t words = (uint32_t)(lds / 4);
    const bool few = blocks_occ / (kOrdStretch / kStretch) <= kOrdFew;
    if (few) (small ? k_order<false, 1024> : k_order<true, 1024>)<<<l.dim, 1024, lds, stream>>>(dm, dl, l.grid, words);
    else (small ? k_order<false, 512> : k_order<true, 512>)<<<l.dim, 512, lds, stream>>>(dm, dl, l.grid, words);
  }
  {
    const size_t lds = ((size_t)maxB * 3 + 1) * 64 * 4 + ((size_t)maxB * 3 + 1 + maxE) * 4;
    const Launch l = all_progs(blocks(maxW, 64));
    if (maxB <= kRegBlocks) k_fixpoint_regs<<<l.dim, 64, 0, stream>>>(dm, dl, l.grid);
    else if (lds <= 64 * 1024) k_fixpoint<true><<<l.dim, 64, lds, stream>>>(dm, dl, l.grid);
    else k_fixpoint<false><<<l.dim, 64, 0, stream>>>(dm, dl, l.grid);
  }
  static_assert(kEvtThreads == kStretch && kStretch == 256, "the block map counts stretches of 256 entries");
  if (blocks_occ) k_events<<<(uint32_t)blocks_occ, kEvtThreads, 0, stream>>>(dm, dl, map_occ);
  const StageGrid g_count = {maxT, blocks(maxB, 4), blocks(maxN, TB * kStageReps)};
  const Launch l_count = all_progs(g_count.a + g_count.b + g_count.c);
  k_stage_count<<<l_count.dim, 256, (size_t)maxW * 4, stream>>>(dm, dl, l_count.grid, g_count);
  if (maxW <= kTileWords && maxT <= kTileCounts) {
    k_stage_scan<true><<<dim3(1, n), 1024, 0, stream>>>(dm, dl);
  } else {
    k_stage_scan<false><<<dim3(1 + blocks(maxW, kTileWords), n), 1024, 0, stream>>>(dm, dl);
    k_seed_count<<<dim3(blocks(maxT, 4), n), 256, 0, stream>>>(dm, dl);
    k_scan<kScanSeed><<<n, 1024, 0, stream>>>(dm, dl);
  }
  e = hipGetLastError();
  if (e != hipSuccess) return fail(hip_fail(e));
  if (!known) {
    k_collect<<<(n + 63) / 64, 64, 0, stream>>>(dm, dl, n);
    e = hipMemcpyAsync(batch->host_counters, a1 + o_counters, (size_t)n * kCounters * 4, hipMemcpyDeviceToHost, stream);
    if (e == hipSuccess) e = hipStreamSynchronize(stream);
    if (e != hipSuccess) return fail(hip_fail(e));
    for (uint32_t k = 0; k < n; ++k)
      if (batch->host_counters[(size_t)k * kCounters + kCtrNotStrict]) return fail(VL_E_NOT_STRICT);
    batch->sizes.resize((size_t)n * 3);
    for (uint32_t k = 0; k < n; ++k) {
      const uint32_t *c = batch->host_counters + (size_t)k * kCounters;
      batch->sizes[3 * k] = c[kCtrPlanLen]; batch->sizes[3 * k + 1] = c[kCtrSeg]; batch->sizes[3 * k + 2] = c[kCtrSeed];
    }
    const int32_t rc2 = layout2();
    if (rc2 != VL_OK) return fail(rc2);
    placed(h, batch->stage_b);
    e = hipMemcpyAsync(a1 + o_lives, batch->stage_b, (size_t)n * sizeof(DevLive), hipMemcpyHostToDevice, stream);
    if (e != hipSuccess) return fail(hip_fail(e));
  }
  const uint32_t per_a = blocks(maxT, 4);
  const uint32_t in_rows = (n + 7) / 8 * 8;   // programs with those that fill up the last row of eight
  const Grid in_dies = {n, batch->dealt && (uint64_t)per_a * in_rows <= kDealtBlocks ? 3u : 0u};
  const StageGrid g_fill = {per_a * (in_dies.dealt ? in_rows : n), (uint32_t)blocks_instr, (uint32_t)blocks_occ};
  const StageGrid g_fin = {blocks(maxB, 4), blocks(maxT, TB), blocks(max_seed, TB)};
  k_stage_fill<<<g_fill.a + g_fill.b + g_fill.c, 256, 0, stream>>>(dm, dl, in_dies, g_fill, per_a, map_instr, map_occ);
  // dense points go along where they are few workgroups, as many as the device takes at once; where they are
  // many, a launch more is nothing beside them
  const uint32_t across = (maxW + 63) / 64;
  const bool dense_along = dense && (uint64_t)across * maxT * n <= 1024;
  const uint32_t n_dense = dense_along ? across * maxT : 0u;
  const Launch l_fin = all_progs(n_dense + g_fin.a + g_fin.b + g_fin.c + blocks(maxV + 1, TB));
  (dense_along ? k_stage_finish<true> : k_stage_finish<false>)<<<l_fin.dim, 256, 0, stream>>>(dm, dl, l_fin.grid, g_fin, n_dense, across);
  if (dense && !dense_along) {
    k_dense<<<dim3((maxW + 63) / 64, maxT, n), 256, 0, stream>>>(dm, dl);
  }
  e = hipGetLastError();
  if (e != hipSuccess) return fail(hip_fail(e));

  // ---- handles ----
  if (fresh) {
    batch->lives.resize(n);
    for (uint32_t k = 0; k < n; ++k) {
      vl_live *l = new (std::nothrow) vl_live;
      if (!l) {
        for (uint32_t j = 0; j < k; ++j) delete batch->lives[j];
        batch_free(batch);
        return VL_E_SHAPE;
      }
      l->batch = batch; l->index = k; l->mir = mirs[k]; l->magic = kLiveMagic;
      batch->lives[k] = l;
    }
    batch->refs = n;
  }
  for (uint32_t k = 0; k < n; ++k) {
    vl_live *l = batch->lives[k];
    l->h = h[k];
    l->dev = batch->dev_lives + place[k];
    l->span = span;
    live[k] = l;
  }
  batch->uploaded.assign((const char *)h.data(), (const char *)h.data() + (size_t)n * sizeof(DevLive));
  batch->sized = true;
  batch->sized_tile_len = tile_len;
  batch->sized_dense = dense;
  return VL_OK;
}

extern "C" int32_t vl_liveness(const vl_mir *mir, uint32_t flags, vl_stream stream, vl_live **live) {
  if (!live) return VL_E_NULL;
  return vl_liveness_multi(&mir, 1, flags, 0, stream, live);
}

extern "C" int32_t vl_live_get(const vl_live *l, vl_live_view *v) {
  if (!l || !v) return VL_E_NULL;
  if (l->magic != kLiveMagic) return VL_E_ARG;
  const DevMir &m = l->mir->h;
  v->n_instr = m.N; v->n_vreg = m.V; v->n_block = m.B; v->n_occ = m.O; v->words = m.W;
  v->n_seg = l->h.n_seg; v->n_tile = l->h.T; v->tile_len = l->h.tile_len;
  v->plan_len = l->h.plan_len + m.O;   // occupancy events + one check per occurrence
  v->sweeps = l->batch->host_counters[(size_t)l->index * kCounters + kCtrSweeps];
  v->live_in = (const uint32_t *)l->h.live_in; v->live_out = (const uint32_t *)l->h.live_out;
  v->live_after = (const uint32_t *)l->h.live_after; v->occ_kill = (const uint8_t *)l->h.occ_kill;
  v->seg_off = (const uint32_t *)l->h.seg_off; v->seg = (const uint32_t *)l->h.seg; v->hull = (const uint32_t *)l->h.hull;
  return VL_OK;
}
