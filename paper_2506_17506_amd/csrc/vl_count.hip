// All violations of each candidate instead of the first (Section 4.5 sorts the model's
// failures into dataflow and hardware-constraint violations; Section 6 proposes the
// verifier as feedback or reward).  With T(v) = the register of v's first occurrence:
//   n_cons  occurrences whose register differs from T(their vreg)
//   n_real  mentioned vregs whose T(v) breaks a hardware rule, real_bits the rules broken
//   n_safe  pairs of one class that are in some P(i) together and whose tuples overlap
// The pairs (the interference relation) depend on the program only: they are enumerated
// once per program from the live intervals and kept with the program handle.
#include <algorithm>
#include <cstring>
#include <mutex>
#include <utility>
#include <vector>

#include "vl_dev.h"

using namespace vl;

namespace {

// ---- interference pairs ------------------------------------------------------------------
// do the interval lists [a0, a1) and [b0, b1) of `seg` (ascending runs [start, end)) share a point?
__device__ inline bool lists_meet(const uint32_t VL_GLOBAL *seg, uint32_t a0, uint32_t a1, uint32_t b0, uint32_t b1) {
  uint32_t x = a0, y = b0;
  while (x < a1 && y < b1) {
    const uint32_t xs = seg[2 * (size_t)x], xe = seg[2 * (size_t)x + 1], ys = seg[2 * (size_t)y], ye = seg[2 * (size_t)y + 1];
    if (max(xs, ys) < min(xe, ye)) return true;
    if (xe <= ye) ++x; else ++y;
  }
  return false;
}

// The pairs (a, b), a < b, are kept as records of eight words, a and up to seven of its partners,
// each vreg with its width in the upper byte (vreg numbers stay below 2^24: VL_MAX_VREG); unused
// places hold a vreg of width 0, which overlaps nothing.  (Records instead of pairs: what is
// looked up for a is looked up once for seven pairs, and a pair takes 4.6 bytes instead of 8.)
constexpr uint32_t kPartners = 7;

// One wavefront per vreg a, its lanes striding over b > a; blockIdx.y = program.  kFill = false:
// cnt[a] = number of records; kFill = true: the records are written from off[a] on, in ascending b.
// Vregs are taken 64 at a time, and a group whose hulls taken together ([earliest start, latest
// end), from k_hull_groups) miss a's hull is passed over: vregs are mostly numbered in the
// order they are first written, so most groups lie entirely before or after a.
struct PairJob {
  const DevMir *mir;
  const DevLive *live;
  uint32_t *cnt;         // [V]
  const uint64_t *off;   // [V]
  uint32_t *records;     // [n_records][8]: vreg | width << 24
  uint2 *groups;         // [(V + 63) / 64] (earliest start, latest end) of the group's non-empty hulls
};

// one wavefront per group of 64 vregs
__global__ __launch_bounds__(256) void k_hull_groups(const PairJob *__restrict__ jobs) {
  const PairJob &J = jobs[blockIdx.y];
  const DevMir VL_GLOBAL &m = *as_global(J.mir);
  const DevLive VL_GLOBAL &L = *as_global(J.live);
  const uint32_t lane = threadIdx.x & 63u, g = blockIdx.x * 4 + (threadIdx.x >> 6);
  if ((size_t)g * 64 >= m.V) return;
  const uint32_t v = g * 64 + lane;
  uint32_t lo = 0xFFFFFFFFu, hi = 0;
  if (v < m.V && L.hull[2 * (size_t)v + 1] != 0) { lo = L.hull[2 * (size_t)v]; hi = L.hull[2 * (size_t)v + 1]; }   // (0, 0): never in any P(i)
  for (int d = 32; d >= 1; d >>= 1) {
    lo = min(lo, (uint32_t)__shfl_xor((int)lo, d, 64));
    hi = max(hi, (uint32_t)__shfl_xor((int)hi, d, 64));
  }
  if (lane == 0) J.groups[g] = make_uint2(lo, hi);
}

// off[a] = number of records of the vregs below a, totals[program] = all of them: one workgroup
// per program, a contiguous run of vregs per thread
__global__ __launch_bounds__(1024) void k_pair_offsets(const PairJob *__restrict__ jobs, uint64_t *__restrict__ totals) {
  const PairJob &J = jobs[blockIdx.x];
  const uint32_t V = as_global(J.mir)->V;
  uint64_t *off = const_cast<uint64_t *>(J.off);   // written here, read by the filling launch
  __shared__ uint64_t part[16];
  const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
  const uint32_t per = (V + 1023u) / 1024u, lo = min(V, threadIdx.x * per), hi = min(V, lo + per);
  uint64_t mine = 0;
  for (uint32_t a = lo; a < hi; ++a) mine += J.cnt[a];
  uint64_t incl = mine;
  for (int d = 1; d < 64; d <<= 1) {
    const uint64_t y = __shfl_up(incl, d, 64);
    if ((int)lane >= d) incl += y;
  }
  if (lane == 63) part[wave] = incl;
  __syncthreads();
  uint64_t run = incl - mine, total = 0;
  for (uint32_t k = 0; k < 16; ++k) {
    if (k < wave) run += part[k];
    total += part[k];
  }
  for (uint32_t a = lo; a < hi; ++a) { off[a] = run; run += J.cnt[a]; }
  if (threadIdx.x == 0) totals[blockIdx.x] = total;
}

template <bool kFill>
__global__ __launch_bounds__(256) void k_pairs(const PairJob *__restrict__ jobs) {
  const PairJob &J = jobs[blockIdx.y];
  const DevMir VL_GLOBAL &m = *as_global(J.mir);
  const DevLive VL_GLOBAL &L = *as_global(J.live);
  const uint32_t lane = threadIdx.x & 63u, a = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (a >= m.V) return;   // whole wavefronts leave; nothing below synchronises the workgroup
  const uint32_t h0 = L.hull[2 * (size_t)a], h1 = L.hull[2 * (size_t)a + 1];
  const uint32_t s0 = L.seg_off[a], s1 = L.seg_off[a + 1], cls = attr_class(m.vattr[a]), width_a = attr_width(m.vattr[a]);
  uint32_t VL_GLOBAL *const records = kFill ? as_global_rw(J.records) + 8 * J.off[a] : nullptr;
  uint32_t n = 0;   // partners so far
  auto place = [](uint32_t x) { return x / kPartners * 8u + 1u + x % kPartners; };   // of the x-th partner
  const uint32_t n_groups = (m.V + 63u) / 64u;
  for (uint32_t g0 = a / 64; g0 < n_groups; g0 += 64) {   // 64 groups at a time, one per lane
    uint2 span = make_uint2(0xFFFFFFFFu, 0u);
    if (g0 + lane < n_groups) span = J.groups[g0 + lane];
    uint64_t todo = __ballot(span.x < h1 && h0 < span.y);
    while (todo) {
      const uint32_t b = (g0 + (uint32_t)__builtin_ctzll(todo)) * 64 + lane;
      todo &= todo - 1;
      bool hit = false;
      const uint32_t attr_b = b > a && b < m.V ? m.vattr[b] : 0u;
      if (b > a && b < m.V && attr_class(attr_b) == cls && L.hull[2 * (size_t)b] < h1 && h0 < L.hull[2 * (size_t)b + 1])
        hit = lists_meet(L.seg, s0, s1, L.seg_off[b], L.seg_off[b + 1]);
      const uint64_t hits = __ballot(hit);
      if (kFill && hit) records[place(n + __popcll(hits & ((1ull << lane) - 1ull)))] = b | (attr_width(attr_b) << 24);
      n += __popcll(hits);
    }
  }
  const uint32_t n_records = (n + kPartners - 1) / kPartners;
  if (!kFill && lane == 0) J.cnt[a] = n_records;
  if (kFill) {
    for (uint32_t r = lane; r < n_records; r += 64) records[8 * r] = a | (width_a << 24);
    if (lane < kPartners && n + lane < n_records * kPartners) records[place(n + lane)] = 0;
  }
}

// ---- per call ----------------------------------------------------------------------------
// A sample without any violation has all counts zero, and the verifier's walk finds those at a
// fraction of the cost of counting (it tests a definition against what is occupied, not against
// every value it interferes with).  So a call runs the walk first, lists each job's failed samples
// (k_cnt_list) and counts only those (k_cnt_rows).
struct DevCountJob {
  const DevMir *mir;
  const DevLive *live;
  const uint16_t *cand;
  vl_counts *out;
  const vl_result *verdicts;   // [K] of the walk; the pairs of safety violations are not in them
  const uint32_t *records;     // [n_records][8]: the interfering pairs
  uint64_t ld, n_records;
  uint32_t K, fail_base, wide, table;   // fail_base: first entry in the list of failed samples; wide: rows can be read 16 bytes
                                        // at a time; table: where the table of registers fits (kTableFour and on)
  float records_per_few;                // of a part, for every few samples that failed (parts_of)
};
struct Unit { uint32_t job_n, first, part, parts; };   // samples failed[first .. first + n) of a job (job | n << 16), a share of its work
struct Head { uint32_t n_units, taken, pad[62]; };     // of a launch; travel with the job table, zeroed by it
// Tables of the registers of four samples, 8 bytes per vreg, in LDS; of two samples, 4 bytes, in LDS; of four samples in
// memory.  (17 programs, one of them of 22,500 vregs, 100 samples each, all failing: 252 us with that one's tables in memory, 192
// with two samples in LDS; alone 132 and 80.)
enum { kTableFour = 0, kTableTwo = 1, kTableMemory = 2 };
__host__ __device__ constexpr uint32_t at_once(uint32_t table) { return table == kTableTwo ? 2u : 4u; }   // samples per workgroup
__host__ __device__ constexpr uint32_t launch_of(uint32_t table) { return table == kTableMemory ? 1u : 0u; }
constexpr uint32_t kLaunches = 2;   // with tables in LDS, and in memory
struct UnitLists { Unit *of[kLaunches]; };

constexpr size_t kTableBytes = 152 * 1024;       // of a compute unit's 160 KB
constexpr uint32_t kLeastRecords = 8192;         // of a part: with fewer, filling the table takes longer than the pairs
constexpr uint32_t kMostRecords = 1u << 22;      // keeps a lane's counts (7 pairs of a record, twice that many, 1,024 lanes) below 2^16
constexpr uint32_t kRounds = 3;                  // units per workgroup, about, so that workgroups end together (one job: all alike, one)

// How many parts a program's pairs are cut into when `fews` fours (twos) of its samples failed.  Every part fills the table
// anew, so there are as many as give every workgroup of the launch work, and no more: a job takes its share of
// the launch (its share of all records, once per four samples), and the fewer samples failed the more parts it is.
__device__ inline uint32_t parts_of(const DevCountJob &J, uint32_t fews) {
  const float share = min(J.records_per_few * (float)fews, (float)kMostRecords);
  if (share < (float)kLeastRecords) return (uint32_t)max((J.n_records + kLeastRecords - 1) / kLeastRecords, (uint64_t)1);
  return (uint32_t)max(J.n_records / (uint64_t)share, (uint64_t)1);   // (rounded down: a last round for a few units costs more)
}

// One wavefront per job: clears the counts, lists the failed samples and the units of work they make.
__global__ __launch_bounds__(256) void k_cnt_list(const DevCountJob *__restrict__ jobs, uint32_t n_jobs, Head *heads, uint32_t *__restrict__ failed,
                                                  const UnitLists units) {
  const uint32_t lane = threadIdx.x & 63u, j = blockIdx.x * 4u + (threadIdx.x >> 6);
  if (j >= n_jobs) return;
  const DevCountJob &J = jobs[j];
  uint32_t n = 0;
  constexpr uint32_t kAhead = 4;   // reads of verdicts in flight
  for (uint32_t k0 = 0; k0 < J.K; k0 += 64 * kAhead) {
    uint32_t status[kAhead];
#pragma unroll
    for (uint32_t u = 0; u < kAhead; ++u) {
      const uint32_t k = k0 + u * 64 + lane;
      status[u] = k < J.K ? J.verdicts[k].status : (uint32_t)VL_STATUS_OK;
    }
#pragma unroll
    for (uint32_t u = 0; u < kAhead; ++u) {
      const uint32_t k = k0 + u * 64 + lane;
      const bool bad = status[u] != VL_STATUS_OK;
      if (k < J.K) J.out[k] = vl_counts{0, 0, 0, 0, 0, {0, 0, 0}};
      const uint64_t which = __ballot(bad);
      if (bad) failed[J.fail_base + n + __popcll(which & ((1ull << lane) - 1ull))] = k;
      n += (uint32_t)__popcll(which);
    }
  }
  if (!n) return;
  const uint32_t per = at_once(J.table), fews = (n + per - 1) / per, parts = parts_of(J, fews), mine = fews * parts;
  uint32_t at = 0;
  if (lane == 0) at = __hip_atomic_fetch_add(&heads[launch_of(J.table)].n_units, mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  at = __builtin_amdgcn_readfirstlane(at);
  Unit *const list = launch_of(J.table) ? units.of[1] : units.of[0];
  for (uint32_t x = lane; x < mine; x += 64) {
    const uint32_t few = x / parts;
    list[at + x] = Unit{j | (min(per, n - few * per) << 16), J.fail_base + few * per, x % parts, parts};
  }
}

// A workgroup takes a unit: up to four failed samples of a job and a share of the job's
// occurrences, vregs and pairs.  The registers T of the four samples' first occurrences are
// gathered into LDS, 8 bytes per vreg (u16 x 4), and everything is counted against that table, the
// four samples at once in packed 16-bit arithmetic:
//   consistency     eight occurrences per lane: their vregs (32 bytes, shared by the samples) and
//                   registers (16 bytes per sample), one 8-byte LDS read per occurrence
//   realizability   as the table is filled
//   safety          a record of seven pairs per lane, eight LDS reads; with u = max(pa - pb, 0) and
//                   v = max(pb - pa, 0) the tuples overlap iff u < width(b) and v < width(a),
//                   exact in saturating arithmetic for any 16-bit register
// What bounds it: the vector instructions of the pairs (18 per pair and four samples) and their
// LDS reads.  The pairs of a large program (600,000 for 20,000 instructions) are cut into parts, so
// that a few failed samples still make work for the whole device; each part fills
// the table anew, which costs as much as some 8,192 records, so there are no more than needed (parts_of).
// Units are taken as workgroups get free.  (64 programs x 100 samples, us per call; parts of 8,192 records
// whatever failed: a fifth fails 224, half 338, all 507; as here 214, 299, 415.  A table in memory for all
// samples, [vreg][sample], with a pass each for table, consistency and safety, took 428 whatever failed.)
template <uint32_t kTable>
__device__ __attribute__((always_inline)) inline void count_unit(const Unit &W, const DevCountJob &J, const uint32_t *failed, uint2 *table_at, uint32_t (&sums)[4][4]) {
  constexpr uint32_t kAtOnce = at_once(kTable), kHalf = kAtOnce / 2;
  struct alignas(4 * kHalf) Regs { uint32_t two[kHalf]; };   // of a vreg, two samples in a word
  Regs *const table = (Regs *)table_at;
  typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
  auto both = [](uint32_t x) { return __builtin_bit_cast(u16x2, x); };
  // 1 in both halves, in a form the compiler cannot see through: a minimum with a known 1 is
  // turned into two compares and a merge instead of one packed instruction
  u16x2 one;
  asm volatile("v_mov_b32 %0, 0x10001" : "=v"(one));
  const uint32_t tid = threadIdx.x, lane = tid & 63u, n_samples = W.job_n >> 16;
  const DevMir VL_GLOBAL &m = *as_global(J.mir);
  const DevLive VL_GLOBAL &L = *as_global(J.live);
  const uint16_t VL_GLOBAL *row[kAtOnce];
#pragma unroll
  for (uint32_t c = 0; c < kAtOnce; ++c) row[c] = as_global(J.cand) + (uint64_t)failed[W.first + min(c, n_samples - 1)] * J.ld;   // (past the last: repeated, not counted)
  if (tid < kAtOnce * 4) (&sums[0][0])[tid] = 0;
  uint32_t n_real[kAtOnce] = {}, rules[kAtOnce] = {};
  // the table; this part's share of the vregs is tested against the hardware rules
  const uint32_t v_lo = (uint32_t)((uint64_t)m.V * W.part / W.parts), v_hi = (uint32_t)((uint64_t)m.V * (W.part + 1) / W.parts);
  for (uint32_t v0 = tid; v0 < m.V; v0 += 4 * 1024) {
    uint32_t f[4], p[4][kAtOnce];
#pragma unroll
    for (uint32_t t = 0; t < 4; ++t) f[t] = v0 + t * 1024 < m.V ? L.first[v0 + t * 1024] : kNone;
#pragma unroll
    for (uint32_t t = 0; t < 4; ++t)
#pragma unroll
      for (uint32_t c = 0; c < kAtOnce; ++c) p[t][c] = f[t] != kNone ? row[c][f[t]] : 0u;
#pragma unroll
    for (uint32_t t = 0; t < 4; ++t) {
      const uint32_t v = v0 + t * 1024;
      if (v >= m.V) break;
      Regs r;
#pragma unroll
      for (uint32_t h = 0; h < kHalf; ++h) r.two[h] = p[t][2 * h] | (p[t][2 * h + 1] << 16);
      table[v] = r;
      if (f[t] == kNone || v < v_lo || v >= v_hi) continue;
      const uint32_t attr = m.vattr[v];
#pragma unroll
      for (uint32_t c = 0; c < kAtOnce; ++c) {
        const uint32_t bad = bad_bits(m, attr, p[t][c]);
        n_real[c] += bad != 0;
        rules[c] |= bad;
      }
    }
  }
  __syncthreads();
  // consistency
  u16x2 n_stray2[kHalf] = {}, n_pair2[kHalf] = {};
  auto stray = [&](uint32_t v, const uint32_t (&p)[kHalf]) __attribute__((always_inline)) {
    const Regs t = table[v];
#pragma unroll
    for (uint32_t h = 0; h < kHalf; ++h) n_stray2[h] += __builtin_elementwise_min(both(p[h] ^ t.two[h]), one);
  };
  auto stray_at = [&](uint32_t o) __attribute__((always_inline)) {
    uint32_t p[kHalf];
#pragma unroll
    for (uint32_t h = 0; h < kHalf; ++h) p[h] = row[2 * h][o] | ((uint32_t)row[2 * h + 1][o] << 16);
    stray(m.occ_vreg[o], p);
  };
  {
    const uint32_t pieces = m.O / 8u;   // whole pieces of eight occurrences; the rest is looked at one by one
    const uint32_t lo = (uint32_t)((uint64_t)pieces * W.part / W.parts), hi = (uint32_t)((uint64_t)pieces * (W.part + 1) / W.parts);
    if (J.wide) {
      for (uint32_t x = lo + tid; x < hi; x += 1024) {
        u32x4 r[kAtOnce];
#pragma unroll
        for (uint32_t c = 0; c < kAtOnce; ++c) r[c] = *reinterpret_cast<const u32x4 VL_GLOBAL *>(row[c] + 8u * x);
        const u32x4 va = *reinterpret_cast<const u32x4 VL_GLOBAL *>(m.occ_vreg + 8u * x), vb = *reinterpret_cast<const u32x4 VL_GLOBAL *>(m.occ_vreg + 8u * x + 4u);
#pragma unroll
        for (uint32_t t = 0; t < 8; ++t) {
          const uint32_t half = t & 1u ? 0x07060302u : 0x05040100u;   // the t-th register of two samples, side by side
          uint32_t p[kHalf];
#pragma unroll
          for (uint32_t h = 0; h < kHalf; ++h) p[h] = __builtin_amdgcn_perm(r[2 * h + 1][t / 2], r[2 * h][t / 2], half);
          stray(t < 4 ? va[t & 3] : vb[t & 3], p);
        }
      }
    } else {
      for (uint32_t o = 8u * lo + tid; o < 8u * hi; o += 1024) stray_at(o);
    }
    if (W.part == 0)
      for (uint32_t o = 8u * pieces + tid; o < m.O; o += 1024) stray_at(o);
  }
  // safety
  {
    const uint64_t e_lo = J.n_records * W.part / W.parts, e_hi = J.n_records * (W.part + 1) / W.parts;
    const u32x4 VL_GLOBAL *records = (const u32x4 VL_GLOBAL *)(uintptr_t)(J.records) + 2 * e_lo;
    const uint32_t n = (uint32_t)(e_hi - e_lo);
    auto at = [&](uint32_t x) { return table[x & 0xFFFFFFu]; };
    auto width2 = [&](uint32_t x) { return both(__builtin_amdgcn_perm(x, x, 0x0C030C03u)); };   // in both halves
    auto overlap = [&](u16x2 ra, u16x2 rb, u16x2 wa, u16x2 wb) __attribute__((always_inline)) {
      const u16x2 x = __builtin_elementwise_sub_sat(ra, rb), y = __builtin_elementwise_sub_sat(rb, ra);
      return __builtin_elementwise_min(__builtin_elementwise_min(__builtin_elementwise_sub_sat(wb, x), __builtin_elementwise_sub_sat(wa, y)), one);
    };
    // The next record is in flight while one is looked at, since a compute unit has few wavefronts to look at others
    // meanwhile (64 programs x 100, half failing: 298 -> 292 us a call).  (Attributes read ahead beside it: 200 small programs
    // 235 -> 261.)
    u32x4 next_lo = 0, next_hi = 0;
    if (tid < n) { next_lo = records[2 * tid]; next_hi = records[2 * tid + 1]; }
    for (uint32_t x = tid; x < n; x += 1024) {
      const u32x4 lo = next_lo, hi = next_hi;
      if (x + 1024 < n) { next_lo = records[2 * (x + 1024)]; next_hi = records[2 * (x + 1024) + 1]; }
      const uint32_t b[kPartners] = {lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
      const Regs ta = at(lo.x);
      Regs tb[kPartners];
#pragma unroll
      for (uint32_t t = 0; t < kPartners; ++t) tb[t] = at(b[t]);
      const u16x2 wa = width2(lo.x);
#pragma unroll
      for (uint32_t t = 0; t < kPartners; ++t) {
        const u16x2 wb = width2(b[t]);
#pragma unroll
        for (uint32_t h = 0; h < kHalf; ++h) n_pair2[h] += overlap(both(ta.two[h]), both(tb[t].two[h]), wa, wb);
      }
    }
  }
#pragma unroll
  for (uint32_t c = 0; c < kAtOnce; ++c) {
    uint32_t s[3] = {n_stray2[c / 2][c % 2], n_real[c], n_pair2[c / 2][c % 2]}, bits = rules[c];
    for (int d = 32; d >= 1; d >>= 1) {
#pragma unroll
      for (uint32_t t = 0; t < 3; ++t) s[t] += (uint32_t)__shfl_xor((int)s[t], d, 64);
      bits |= (uint32_t)__shfl_xor((int)bits, d, 64);
    }
    if (lane == 0) {
#pragma unroll
      for (uint32_t t = 0; t < 3; ++t)
        if (s[t]) atomicAdd(&sums[c][t], s[t]);
      if (bits) atomicOr(&sums[c][3], bits);
    }
  }
  __syncthreads();
  if (tid < n_samples) {
    vl_counts VL_GLOBAL *out = as_global_rw(J.out) + failed[W.first + tid];
    const uint32_t strays = sums[tid][0], unreal = sums[tid][1], overlaps = sums[tid][2];
    if (strays) atomicAdd(&out->n_cons, strays);
    if (unreal) { atomicAdd(&out->n_real, unreal); atomicOr(&out->real_bits, sums[tid][3]); }
    if (overlaps) atomicAdd(&out->n_safe, overlaps);
    const uint32_t kinds = (strays ? 1u : 0u) | (unreal ? 2u : 0u) | (overlaps ? 4u : 0u);
    if (kinds) atomicOr(&out->kinds, kinds);
  }
}

// kLds = false: the tables lie in memory, `max_v` vregs of four samples for each workgroup
template <bool kLds>
__global__ __launch_bounds__(1024) void k_cnt_rows(const DevCountJob *__restrict__ jobs, Head *head, const uint32_t *__restrict__ failed,
                                                   const Unit *__restrict__ units, uint2 *tables, uint32_t max_v) {
  extern __shared__ uint2 table_lds[];   // [V]
  __shared__ uint32_t sums[4][4];        // per sample: strays, unrealizable vregs, overlapping pairs, rules broken
  __shared__ uint32_t taken;
  const uint32_t n_units = head->n_units;
  for (;;) {
    if (threadIdx.x == 0) taken = __hip_atomic_fetch_add(&head->taken, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    const uint32_t u = __builtin_amdgcn_readfirstlane(taken);
    if (u >= n_units) break;   // (every workgroup gets here: the counter only grows)
    const Unit W = units[u];
    const DevCountJob &J = jobs[W.job_n & 0xFFFFu];
    if (!kLds) count_unit<kTableMemory>(W, J, failed, tables + (size_t)blockIdx.x * max_v, sums);
    else if (J.table == kTableTwo) count_unit<kTableTwo>(W, J, failed, table_lds, sums);
    else count_unit<kTableFour>(W, J, failed, table_lds, sums);
    __syncthreads();   // table and sums are reused by the next unit
  }
}

// Workspaces of a device, used in turn, so that a call waits only for the one kWorkspaces calls ago.
constexpr uint32_t kWorkspaces = 4;
constexpr size_t kHeads = kLaunches * sizeof(Head);
struct Work {
  char *dev = nullptr, *host = nullptr;   // Head and job table; host: pinned
  uint32_t cap = 0;                       // jobs
  char *mem = nullptr;                    // verdicts, failed samples, units, tables that do not fit LDS
  size_t mem_cap = 0;
  WalkSpace walk;                         // job table and board of the walk: a stream's own stay as its verifications left them
  hipEvent_t consumed = nullptr;          // recorded after the last kernel of a call
  bool in_flight = false;
};
struct Works {
  std::mutex mu;
  Work one[kWorkspaces];
  uint32_t turn = 0;
};
Works g_works[16];

// Enumerates the interference pairs of the programs that do not have them yet, from the
// intervals of their analyses (which must be complete or enqueued on `stream`): one counting
// launch over all of them, the offsets summed per program on the device, one filling launch.  Synchronises
// the stream twice.
int32_t build_pairs(const std::vector<std::pair<vl_mir *, const vl_live *>> &todo, hipStream_t stream) {
  const size_t n = todo.size();
  size_t total_v = 0;
  uint32_t max_v = 0;
  std::vector<size_t> base(n);
  for (size_t j = 0; j < n; ++j) {
    base[j] = total_v;
    total_v += todo[j].first->h.V;
    max_v = std::max(max_v, todo[j].first->h.V);
  }
  if (total_v == 0) {
    for (auto &t : todo) { t.first->edges = nullptr; t.first->n_edges = 0; t.first->edges_built = true; }
    return VL_OK;
  }
  // device scratch: counts, offsets, the job table; host: the same, pageable (copies wait for the stream)
  uint32_t *cnt = nullptr;
  uint64_t *off = nullptr;
  uint2 *groups = nullptr;
  uint64_t *totals_dev = nullptr;
  PairJob *jobs_dev = nullptr;
  void *all_pairs = nullptr;   // one allocation for the pairs of every program of this call, handed to them on success
  auto cleanup = [&]() { (void)hipFree(cnt); (void)hipFree(off); (void)hipFree(groups); (void)hipFree(totals_dev); (void)hipFree(jobs_dev); };
  auto fail = [&](hipError_t err) {
    cleanup();
    (void)hipFree(all_pairs);
    return hip_fail(err);
  };
  // (a kernel's groups start at base / 64 + its index: at most one entry per kernel is left unused)
  hipError_t e = device_alloc((void **)&cnt, total_v * 4);
  if (e == hipSuccess) e = device_alloc((void **)&off, total_v * 8);
  if (e == hipSuccess) e = device_alloc((void **)&groups, (total_v / 64 + n + 1) * sizeof(uint2));
  if (e == hipSuccess) e = device_alloc((void **)&totals_dev, n * 8);
  if (e == hipSuccess) e = device_alloc((void **)&jobs_dev, n * sizeof(PairJob));
  if (e != hipSuccess) return fail(e);
  std::vector<PairJob> jobs(n);
  for (size_t j = 0; j < n; ++j)
    jobs[j] = PairJob{todo[j].first->dev, todo[j].second->dev, cnt + base[j], off + base[j], nullptr, groups + base[j] / 64 + j};
  e = hipMemcpyAsync(jobs_dev, jobs.data(), n * sizeof(PairJob), hipMemcpyHostToDevice, stream);
  if (e != hipSuccess) return fail(e);
  const dim3 grid((max_v + 3) / 4, (uint32_t)n);
  k_hull_groups<<<dim3(((max_v + 63) / 64 + 3) / 4, (uint32_t)n), 256, 0, stream>>>(jobs_dev);
  k_pairs<false><<<grid, 256, 0, stream>>>(jobs_dev);
  k_pair_offsets<<<(uint32_t)n, 1024, 0, stream>>>(jobs_dev, totals_dev);
  std::vector<uint64_t> totals(n), first_pair(n);
  e = hipMemcpyAsync(totals.data(), totals_dev, n * 8, hipMemcpyDeviceToHost, stream);
  if (e == hipSuccess) e = hipStreamSynchronize(stream);
  if (e != hipSuccess) return fail(e);
  uint64_t all = 0;
  for (size_t j = 0; j < n; ++j) {
    first_pair[j] = all;
    all += (totals[j] + 7) & ~(uint64_t)7;   // every program's records start on a 256-byte boundary
  }
  if (all) {
    e = device_alloc(&all_pairs, (size_t)all * 32);
    if (e != hipSuccess) return fail(e);
  }
  for (size_t j = 0; j < n; ++j) jobs[j].records = totals[j] ? (uint32_t *)all_pairs + 8 * first_pair[j] : nullptr;
  e = hipMemcpyAsync(jobs_dev, jobs.data(), n * sizeof(PairJob), hipMemcpyHostToDevice, stream);
  if (e == hipSuccess) {
    k_pairs<true><<<grid, 256, 0, stream>>>(jobs_dev);
    e = hipGetLastError();
  }
  if (e == hipSuccess) e = hipStreamSynchronize(stream);   // the host vectors and the scratch go away below
  if (e != hipSuccess) return fail(e);
  cleanup();
  EdgeBlock *block = nullptr;
  if (all_pairs) {
    uint32_t holders = 0;
    for (size_t j = 0; j < n; ++j) holders += totals[j] != 0;
    block = new (std::nothrow) EdgeBlock{all_pairs, {holders}};
    if (!block) { (void)hipFree(all_pairs); return VL_E_SHAPE; }
  }
  for (size_t j = 0; j < n; ++j) {
    todo[j].first->edges = jobs[j].records;
    todo[j].first->n_edges = totals[j];
    todo[j].first->edge_block = totals[j] ? block : nullptr;
    todo[j].first->edges_built = true;
  }
  return VL_OK;
}

}  // namespace

extern "C" int32_t vl_count_violations_multi(const vl_count_job *jobs, uint32_t n_jobs, vl_stream stream_) {
  if (!jobs) return VL_E_NULL;
  if (n_jobs == 0 || n_jobs > 65535) return VL_E_SHAPE;
  for (uint32_t j = 0; j < n_jobs; ++j) {
    const vl_count_job &u = jobs[j];
    if (!u.mir || !u.live || !u.cand || !u.out) return VL_E_NULL;
    if (u.mir->magic != kMirMagic || u.live->magic != kLiveMagic || u.live->mir != u.mir || u.mir->lowered) return VL_E_ARG;
    if (u.K == 0 || u.K > 65535 || u.ld < u.mir->h.O) return VL_E_SHAPE;
  }
  hipStream_t stream = (hipStream_t)stream_;
  int device = 0;
  VL_HIP(hipGetDevice(&device));
  if (device < 0 || device >= 16) return VL_E_ARG;
  Works &all = g_works[device];
  std::lock_guard<std::mutex> lock(all.mu);
  // the pairs of programs seen for the first time (the handle is the cache: not const here)
  {
    std::vector<std::pair<vl_mir *, const vl_live *>> todo;
    for (uint32_t j = 0; j < n_jobs; ++j) {
      vl_mir *mir = const_cast<vl_mir *>(jobs[j].mir);
      if (!mir->edges_built) todo.emplace_back(mir, jobs[j].live);
    }
    // the same program may appear in several jobs
    std::sort(todo.begin(), todo.end(), [](const auto &x, const auto &y) { return x.first < y.first; });
    todo.erase(std::unique(todo.begin(), todo.end(), [](const auto &x, const auto &y) { return x.first == y.first; }), todo.end());
    if (!todo.empty()) {
      const int32_t rc = build_pairs(todo, stream);
      if (rc != VL_OK) return rc;
    }
  }
  // the kernels of the call that last used this workspace must be done with it
  Work &w = all.one[all.turn = (all.turn + 1) % kWorkspaces];
  if (w.in_flight) VL_HIP(hipEventSynchronize(w.consumed));
  w.in_flight = false;
  if (w.cap < n_jobs) {
    if (w.dev) (void)hipFree(w.dev);
    if (w.host) (void)hipHostFree(w.host);
    w.dev = nullptr; w.host = nullptr; w.cap = 0;
    const uint32_t cap = std::max(256u, n_jobs);
    VL_HIP(device_alloc((void **)&w.dev, kHeads + (size_t)cap * sizeof(DevCountJob)));
    VL_HIP(hipHostMalloc((void **)&w.host, kHeads + (size_t)cap * sizeof(DevCountJob), hipHostMallocDefault));
    w.cap = cap;
  }
  if (!w.consumed) VL_HIP(hipEventCreateWithFlags(&w.consumed, hipEventDisableTiming));
  static const bool lds_ok = hipFuncSetAttribute((const void *)k_cnt_rows<true>, hipFuncAttributeMaxDynamicSharedMemorySize, kTableBytes) == hipSuccess;
  auto table_of = [&](const vl_mir *m) -> uint32_t {
    return !lds_ok || m->h.V * sizeof(uint32_t) > kTableBytes ? kTableMemory : m->h.V * sizeof(uint2) > kTableBytes ? kTableTwo : kTableFour;
  };
  // of each launch: the largest table, all records once per few samples, and how many units there can be
  struct Part {
    uint64_t most = 0, least = 0;   // units, with parts as short as they get; with one part for every few samples
    double work = 0;
    size_t table_bytes = 0;
    uint32_t groups = 0;
  } launches[kLaunches];
  uint64_t rows = 0, total_units = 0;
  const uint32_t rounds = n_jobs == 1 ? 1 : kRounds;
  for (uint32_t j = 0; j < n_jobs; ++j) {
    const uint32_t t = table_of(jobs[j].mir);
    Part &p = launches[launch_of(t)];
    const uint64_t fews = (jobs[j].K + at_once(t) - 1) / at_once(t), records = jobs[j].mir->n_edges;
    rows += jobs[j].K;
    p.table_bytes = std::max(p.table_bytes, std::max<size_t>(1, jobs[j].mir->h.V) * 2 * at_once(t));
    p.work += (double)fews * (double)records;
    p.most += fews * std::max<uint64_t>(1, (records + kLeastRecords - 1) / kLeastRecords);
    p.least += fews * (1 + records / kMostRecords) + 1;
  }
  for (uint32_t x = 0; x < kLaunches; ++x) {
    Part &p = launches[x];
    p.groups = x == 0 && p.table_bytes <= kTableBytes / 2 ? 512 : 256;   // workgroups: as many as fit the 256 compute units at once
    p.most = std::min(p.most, p.least + p.groups * rounds);              // (parts_of)
    total_units += p.most;
  }
  if (rows > 0x7FFFFFFFull || total_units > 0x7FFFFFFFull) return VL_E_SHAPE;
  auto up = [](size_t x) { return (x + 255) & ~(size_t)255; };
  const size_t o_failed = up(rows * sizeof(vl_result)), o_units = o_failed + up(rows * 4), o_tables = o_units + up(total_units * sizeof(Unit));
  const size_t bytes = o_tables + (launches[1].most ? launches[1].groups * launches[1].table_bytes : 0);
  if (bytes > w.mem_cap) {
    if (w.mem) (void)hipFree(w.mem);
    w.mem = nullptr; w.mem_cap = 0;
    VL_HIP(device_alloc((void **)&w.mem, bytes));
    w.mem_cap = bytes;
  }
  vl_result *const verdicts = (vl_result *)w.mem;
  uint32_t *const failed = (uint32_t *)(w.mem + o_failed);
  Unit *const units = (Unit *)(w.mem + o_units);
  const UnitLists lists = {{units, units + launches[0].most}};
  Head *const heads = (Head *)w.dev;
  const DevCountJob *const dev_jobs = (const DevCountJob *)(w.dev + kHeads);
  std::vector<vl_job> walk(n_jobs);
  uint32_t at = 0;
  memset(w.host, 0, kHeads);
  for (uint32_t j = 0; j < n_jobs; ++j) {
    const vl_count_job &u = jobs[j];
    DevCountJob &d = ((DevCountJob *)(w.host + kHeads))[j];
    memset(&d, 0, sizeof(d));
    d.mir = u.mir->dev; d.live = u.live->dev; d.cand = u.cand; d.out = u.out; d.verdicts = verdicts + at;
    d.records = (const uint32_t *)u.mir->edges; d.n_records = u.mir->n_edges; d.ld = u.ld; d.K = u.K; d.fail_base = at;
    d.table = table_of(u.mir);
    const Part &p = launches[launch_of(d.table)];
    // (a little more, so that rounding never asks for more units than there is room for)
    d.records_per_few = (float)(1.001 * p.work / ((double)((u.K + at_once(d.table) - 1) / at_once(d.table)) * p.groups * rounds));
    d.wide = ((uintptr_t)u.cand & 15) == 0 && (u.ld & 7) == 0;
    walk[j] = vl_job{u.mir, u.live, u.cand, u.K, u.ld, verdicts + at};
    at += u.K;
  }
  VL_HIP(hipMemcpyAsync(w.dev, w.host, kHeads + (size_t)n_jobs * sizeof(DevCountJob), hipMemcpyHostToDevice, stream));
  const int32_t rc = verdicts_only(walk.data(), n_jobs, stream, w.walk);
  if (rc != VL_OK) {
    (void)hipStreamSynchronize(stream);   // the table's upload
    return rc;
  }
  k_cnt_list<<<(n_jobs + 3) / 4, 256, 0, stream>>>(dev_jobs, n_jobs, heads, failed, lists);
  if (launches[0].most)
    k_cnt_rows<true><<<(uint32_t)std::min<uint64_t>(launches[0].most, launches[0].groups), 1024, launches[0].table_bytes, stream>>>(
        dev_jobs, heads, failed, lists.of[0], nullptr, 0);
  if (launches[1].most)
    k_cnt_rows<false><<<(uint32_t)std::min<uint64_t>(launches[1].most, launches[1].groups), 1024, 0, stream>>>(
        dev_jobs, heads + 1, failed, lists.of[1], (uint2 *)(w.mem + o_tables), (uint32_t)(launches[1].table_bytes / sizeof(uint2)));
  VL_HIP(hipGetLastError());
  VL_HIP(hipEventRecord(w.consumed, stream));
  w.in_flight = true;
  return VL_OK;
}
