// Batched verification of candidate register assignments.
//
// One wavefront handles up to 64 candidates (one per lane) of one kernel over
// one tile of its event stream.  The stream is the same for every candidate
// of a kernel, so it is read once per wavefront, 64 entries at a time, and
// broadcast entry by entry; only the candidate rows differ per lane.
//
//   Consistency   every occurrence is compared with the previous occurrence
//                 of the same vreg (equal along the chain <=> equal to the
//                 first occurrence; the first broken link is the first
//                 inconsistent occurrence).
//   Realizability checked at the first occurrence of each vreg.
//   Safety        per-lane occupancy bitmask per register class in LDS,
//                 [word][lane]; a definition tests its range against the
//                 mask, then sets it; kills clear it.  Tiles start from the
//                 live-in list of their first instruction.
// Each lane keeps the smallest violation key it has seen; tiles combine on a
// board in memory, and the last one to report writes the results.  (Section 3.4 of the paper states the
// three conditions; Section 1 items (1) and (2) define a correct allocation.)
#include <cstring>
#include <mutex>
#include <new>
#include <vector>

#include <type_traits>

#include "../../include/vl_bench.h"
#include "vl_dev.h"

using namespace vl;

namespace vl {
// (Kernel arguments are fetched 64 bytes at a time: with 144 bytes of them for the pair search instead of 120, verification
// of 8 to 64 samples took 0.1 to 0.3 us more.  Hence nothing here that the device does not need.)
struct DevJob {
  const DevMir *mir;
  const DevLive *live;
  const uint16_t *cand;
  vl_result *out;
  uint64_t ld;
  uint32_t K, rows, n_groups, unit_base;
  uint32_t row_base, group_base;   // the job's first entry in Board::keys and Board::arrived
  uint32_t span, n_spans;          // analysis tiles that a workgroup takes at once, and how often that is
  uint8_t transposed;              // cand is [occurrence][candidate]
  uint8_t direct;                  // row-major, aligned, and every row has room for whole chunks up to its pitch
  uint8_t unused[6];               // zero (tables are compared byte by byte)
};
static_assert(sizeof(DevJob) == 80, "no padding");
}  // namespace vl

namespace {

// Occurrences kept per candidate in LDS: three chunks.  A ring slot holds one uint16 per
// candidate row plus padding; its pitch is a compile-time parameter of the walk: 68 (136
// bytes) for up to 64 rows, 52 (104 bytes) for up to 52 rows, e.g. the 50-row halves of 100
// candidates.  With two register classes a workgroup then needs about 31 KB or 25 KB, and
// five or six workgroups share a compute unit's 160 KB.  Both pitches are 2 modulo 8
// dwords, which is what the bank assignment of the staging stores relies on.
constexpr uint32_t kRing = kWalkRing;
constexpr uint32_t kPitchWide = 68, kPitchNarrow = 52;
#ifndef VL_CHECK_WAVES
#define VL_CHECK_WAVES 3
#endif
constexpr uint32_t kCheckWaves = VL_CHECK_WAVES;   // wavefronts per workgroup that stage and check
constexpr uint32_t kWalkThreads = 64 * (1 + kCheckWaves);
constexpr int kStagePasses = (8 + kCheckWaves - 1) / kCheckWaves;
constexpr uint32_t kChunk = kWalkChunk;                 // occurrences staged per step (128 B per row)
constexpr uint32_t kKeyOk = 0xFFFFFFFFu;
constexpr uint32_t kKeyCons = 0u << 28, kKeyReal = 1u << 28, kKeySafe = 2u << 28, kKeyPos = (1u << 28) - 1;

// What the workgroups of one verification share.  Everything is zero before the walk and left
// zero by it, so that no launch is needed to clear it.  Calls that overlap on one board against the rules (their
// counts mix) spoil each other, and what they leave would spoil every later call too.  So where a board can be
// shared at all (WalkSpace::recorded, and the entry point that allocates nothing) the pair search, which follows the
// walk, writes the zeros again: of calls that overlapped, the one whose walk ends last clears what it has in
// common with the others after all of them.
constexpr uint32_t kHeadWords = 64;   // in front of Board::arrived; the first is Launch::finished
struct Board {
  uint32_t *arrived;   // per group of candidate rows: tiles that have reported
  uint32_t *keys;      // per candidate row: ~(smallest violation key so far), 0 = none
};

// The job of unit (or group) x, whose first unit (group) is the field `base` of its entry: 64
// probes at a time, one per lane (two dependent reads for up to 4,096 jobs; a binary search took
// eight for 256).
__device__ inline uint32_t find_job(const DevJob *jobs, uint32_t n_jobs, uint32_t x, uint32_t DevJob::*base) {
  uint32_t lo = 0, len = n_jobs;
  while (len > 1) {
    const uint32_t step = (len + 63u) / 64u, off = __lane_id() * step;
    const uint32_t n = (uint32_t)__popcll(__ballot(off < len && jobs[lo + off].*base <= x));
    lo += (n - 1u) * step;   // bases ascend, and the first probe never lies above x
    len = min(step, len - (n - 1u) * step);
  }
  return lo;
}

// register of occurrence o in candidate k, in either layout
template <class Job> __device__ inline uint32_t cand_at(const Job &J, uint32_t k, uint32_t o) {
  return J.transposed ? J.cand[(uint64_t)o * J.ld + k] : J.cand[(uint64_t)k * J.ld + o];
}

// ---- the candidate walk -----------------------------------------------------------------
// A workgroup of 4 wavefronts takes up to 64 candidate rows of one kernel over one tile
// (a range of instructions).  Occurrences are staged 64 at a time (one 128-byte line per
// row, the next chunk already in flight) into an LDS ring [occurrence % 192][row].  After
// each chunk
//   * one wavefront replays the occupancy events that chunk releases, one candidate per
//     lane, the lane's occupancy mask in LDS as [word][lane];
//   * three wavefronts run the chunk's 64 consistency / realizability checks with one
//     check per lane, looping over their share of the rows: what is uniform per check
//     (ring offsets, class limits) is then computed once per lane instead of once per
//     check and candidate.
// Violations go to a per-row key in LDS (smallest wins) and from there to the board.
// LDS layout (indices into the dynamic shared array, kept as integers so that every
// access is a DS instruction rather than a flat one):
//   [0, occ_words * 64)            occupancy masks [word][lane]
//   [keys, keys + 64)              per-row violation keys
//   [keys + 64, keys + 320)        the occupancy wavefront's event buffer (64 records of 16 bytes)
//   [ring32, ...)                  the ring [occurrence % 192][row], addressed in uint16 from
//                                  ring16 = 2 * ring32; a lane of the check wavefronts reads four
//                                  rows of one occurrence with one 8-byte read
extern __shared__ uint32_t vl_lds[];
#define VL_LDS16 (reinterpret_cast<uint16_t *>(vl_lds))

struct Walk {
  const uint16_t VL_GLOBAL *rows;   // first row of the group
  uint64_t ld;
  uint32_t keys, ring16;  // LDS indices
  // readable occurrences: [max(lo, hi - kWalkReach), hi); hi is the end of the chunk being processed
  uint32_t tid, lane, row, nrows, n_occ, lo, hi;
  uint32_t pre[kStagePasses][5];     // check wavefronts: their share of the chunk being fetched (the fifth word: ragged staging)
  // row-major staging: per pass, this lane's byte offset into the group's rows and its uint16 index into
  // ring slot 0 (kNone in from_row: the pass has no row for this lane)
  uint32_t from_row[kStagePasses], to_ring[kStagePasses];
  int32_t last_piece;   // direct staging: from this lane's piece of a row's first chunk to the last piece with registers, in bytes
};

// Staging is done by the three check wavefronts.  A chunk is 64 rows x 8 pieces of 16 bytes
// (8 occurrences); piece k of row r goes to lane (k, rr) of pass q with
//   r = y + 2 rr + 16 ((k >> 2) ^ u) + 32 z,   q = y + 2 z + 4 u  (0..7),
// the two halves of a 128-byte line (k < 4, k >= 4) belonging to rows 16 apart.  With this
// assignment the 64 lanes of every LDS store below write into 64 different 4-byte words,
// two per bank (slot pitch 34 or 26 dwords, both 2 modulo 8: word = 16 (k & 3) + 8 (row bit
// 4) + rr + const modulo 64), which the 32 banks take in two passes: the least a 64-lane
// store can take.  Check wavefront j takes the passes j, j + 3, j + 6.
__device__ inline uint32_t staged_row(uint32_t lane, uint32_t q) {
  const uint32_t k = lane & 7u, rr = lane >> 3;
  return (q & 1u) + 2u * rr + 16u * ((k >> 2) ^ (q >> 2)) + 32u * ((q >> 1) & 1u);
}

// Occurrence-major candidates, cand[occurrence][candidate] with pitch ld:
// a chunk is then 64 occurrences x 8 pieces of 16 bytes (8 candidates) that already have the
// ring's layout: lane (occurrence o8, piece k) of pass q copies piece k of occurrence
// 8 q + o8, eight lanes reading one 128-byte line.
__device__ inline void load_chunk_occ(Walk &w, uint32_t c0, uint32_t j) {
#pragma unroll
  for (int h = 0; h < kStagePasses; ++h) {
    const uint32_t q = j + kCheckWaves * h;
    w.pre[h][0] = w.pre[h][1] = w.pre[h][2] = w.pre[h][3] = 0;
    if (q >= 8u) continue;
    const uint32_t o = c0 + q * 8u + (w.lane >> 3), piece = w.lane & 7u;
    if (piece * 8u < w.nrows && o < w.n_occ) {   // the 16 bytes lie inside the occurrence's pitch (a multiple of 8)
      const u32x4 x = *reinterpret_cast<const u32x4 VL_GLOBAL *>(w.rows + (uint64_t)o * w.ld + piece * 8u);
      w.pre[h][0] = x.x; w.pre[h][1] = x.y; w.pre[h][2] = x.z; w.pre[h][3] = x.w;
    }
  }
}

// writes the chunk held in registers into the ring as chunk [c0, c0 + 64)
template <uint32_t kRingStride>
__device__ inline void store_chunk_occ(const Walk &w, uint32_t c0, uint32_t j) {
#pragma unroll
  for (int h = 0; h < kStagePasses; ++h) {
    const uint32_t q = j + kCheckWaves * h;
    if (q >= 8u) continue;
    // 8 candidates of one occurrence: two 8-byte stores (ring slots start on 8-byte
    // boundaries); what would fall beyond the slot's pitch is left out
    const uint32_t o = c0 + q * 8u + (w.lane >> 3), piece = w.lane & 7u;
    const uint32_t dst = (w.ring16 + (o % kRing) * kRingStride + piece * 8u) >> 2;   // in 8-byte units
    uint64_t *lds64 = reinterpret_cast<uint64_t *>(vl_lds);
    if (piece * 8u + 4u <= kRingStride) lds64[dst] = (uint64_t)w.pre[h][0] | ((uint64_t)w.pre[h][1] << 32);
    if (piece * 8u + 8u <= kRingStride) lds64[dst + 1] = (uint64_t)w.pre[h][2] | ((uint64_t)w.pre[h][3] << 32);
  }
}

// Direct staging, when every job of the launch allows it (DevJob::direct): without the
// per-lane branches of the general path, a buffer read per pass (descriptor of the group's rows
// in scalar registers, the lane's row offset from set-up) and eight 2-byte stores from an address
// that only needs the chunk's slot added.  Rows past the group's last are never written; their ring
// entries are cleared once at the start.  Beyond the program's last occurrence nothing is read but
// the rest of the 16 bytes it lies in: lanes whose piece lies further repeat that one (a minimum per
// chunk and an addition per pass, which cost nothing that could be measured), and what lands in the
// ring there is never looked at.
__device__ inline void load_chunk_direct(Walk &w, uint32_t c0, __amdgpu_buffer_rsrc_t rows) {
  const int32_t at = min((int32_t)(c0 * 2u), w.last_piece);
#pragma unroll
  for (int h = 0; h < kStagePasses; ++h) {
    if (w.from_row[h] == kNone) continue;
    const u32x4 x = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rows, w.from_row[h] + (uint32_t)at, 0, 0));
    w.pre[h][0] = x.x; w.pre[h][1] = x.y; w.pre[h][2] = x.z; w.pre[h][3] = x.w;
  }
}

template <uint32_t kRingStride>
__device__ inline void store_chunk_direct(const Walk &w, uint32_t c0) {
  const uint32_t slot = (c0 % kRing) * kRingStride;
#pragma unroll
  for (int h = 0; h < kStagePasses; ++h) {
    if (w.from_row[h] == kNone) continue;
    const uint32_t dst = w.to_ring[h] + slot;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      VL_LDS16[dst + (2 * t) * kRingStride] = (uint16_t)w.pre[h][t];
      VL_LDS16[dst + (2 * t + 1) * kRingStride] = (uint16_t)(w.pre[h][t] >> 16);
    }
  }
}

// Ragged staging: rows of any pitch and alignment.  A piece of 8 registers lies in the four or,
// when it starts in the middle of one (bit 0 of from_row), five aligned words around it, which are
// read whole and shifted into place when they are stored.  Each of these words holds part of the
// piece, so nothing beyond the memory's last word is touched as long as the piece is the
// program's; in the chunk that the program ends in, words past the row's last are replaced by that
// one.  (Reading every chunk with 2 bytes per register, verification of 24 programs of
// 1,000-12,000 instructions with 37 packed rows took 81 us, 12 of them before the first chunk; 62 this
// way, 67 with the registers of six wavefronts per SIMD, eleven of which then lie in memory.)
__device__ inline void load_chunk_ragged(Walk &w, uint32_t c0, __amdgpu_buffer_rsrc_t rows, bool shifted) {
#pragma unroll
  for (int h = 0; h < kStagePasses; ++h) {
    if (w.from_row[h] == kNone) continue;
    const uint32_t odd = w.from_row[h] & 1u, at = w.from_row[h] - odd;
    if (c0 + kChunk <= w.n_occ) {
      const u32x4 x = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rows, at, c0 * 2u, 0));
      w.pre[h][0] = x.x; w.pre[h][1] = x.y; w.pre[h][2] = x.z; w.pre[h][3] = x.w;
      if (shifted) w.pre[h][4] = __builtin_amdgcn_raw_buffer_load_b32(rows, at + 12u + 4u * odd, c0 * 2u, 0);
    } else {
      const uint32_t last = (at - (w.lane & 7u) * 16u + 2u * (odd + w.n_occ - 1u)) & ~3u;
#pragma unroll
      for (uint32_t t = 0; t < 5; ++t) w.pre[h][t] = __builtin_amdgcn_raw_buffer_load_b32(rows, min(at + c0 * 2u + 4u * t, last), 0, 0);
    }
  }
}

template <uint32_t kRingStride>
__device__ inline void store_chunk_ragged(const Walk &w, uint32_t c0) {
  const uint32_t slot = (c0 % kRing) * kRingStride;
#pragma unroll
  for (int h = 0; h < kStagePasses; ++h) {
    if (w.from_row[h] == kNone) continue;
    const uint32_t dst = w.to_ring[h] + slot, shift = 16u * (w.from_row[h] & 1u);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const uint32_t x = __builtin_amdgcn_alignbit(w.pre[h][t + 1], w.pre[h][t], shift);
      VL_LDS16[dst + (2 * t) * kRingStride] = (uint16_t)x;
      VL_LDS16[dst + (2 * t + 1) * kRingStride] = (uint16_t)(x >> 16);
    }
  }
}

__device__ inline bool in_ring(const Walk &w, uint32_t o) {
  return o < w.hi && o + kWalkReach >= w.hi && o >= w.lo;
}

// value of occurrence o in this lane's row, from memory
template <bool kT>
__device__ inline uint32_t from_memory(const Walk &w, uint32_t o) {
  return kT ? w.rows[(uint64_t)o * w.ld + w.row] : w.rows[(uint64_t)w.row * w.ld + o];
}

// Waits for the reads of a rare path before it joins the usual one.  The compiler waits where a value
// is used, whichever path it came by, and reads from memory return in order: without this, the usual
// path waited there too, for whatever was fetched ahead (records, rows, the next chunk's checks).
__device__ inline void reads_done() { __builtin_amdgcn_s_waitcnt(0x0070); }   // vmcnt(0) lgkmcnt(0)

template <uint32_t kRingStride, bool kT>
__device__ inline uint32_t fetch(const Walk &w, uint32_t o) {
  if (in_ring(w, o)) return VL_LDS16[w.ring16 + (o % kRing) * kRingStride + w.row];
  return from_memory<kT>(w, o);
}

// Address of the mask word holding register p of a class, and the mask of the tuple.
// The word index is clamped to the class, so a base outside the file cannot leave the
// mask; such a base is reported as unrealizable (or inconsistent), which outranks
// whatever the occupancy test says.
struct Touch { uint32_t addr; uint32_t mlo, mhi; };   // addr: index into the LDS array
__device__ inline Touch locate(const Walk &w, uint32_t attr, uint32_t cls_tab, uint32_t p) {
  const uint32_t width = attr_width(attr);
  const uint32_t F = cls_tab & 0xFFFFu, wbase = cls_tab >> 16;
  const uint32_t last_word = (F - 1u) >> 5;
  const uint32_t word = min(p >> 5, last_word), bitpos = p & 31u;
  const uint32_t wm = width == 32 ? 0xFFFFFFFFu : ((1u << width) - 1u);
  Touch t;
  t.addr = (wbase + word) * 64 + w.lane;
  if (!attr_straddle(attr)) { t.mlo = wm << bitpos; t.mhi = 0; }
  else {
    const uint64_t m64 = (uint64_t)wm << bitpos;
    t.mlo = (uint32_t)m64;
    t.mhi = word < last_word ? (uint32_t)(m64 >> 32) : 0u;
  }
  return t;
}

// Every event flips the bits of its range: an occupy on free bits and a release of held
// bits are both an exclusive-or, exact up to the first clash, which is all that is
// reported.  Returns the bits that were already set (meaningful for occupy-with-test).
__device__ inline uint32_t flip(const Touch &t, bool straddle) {
  uint32_t hit = __hip_atomic_fetch_xor(&vl_lds[t.addr], t.mlo, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) & t.mlo;
  if (straddle) hit |= __hip_atomic_fetch_xor(&vl_lds[t.addr + 64], t.mhi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) & t.mhi;
  return hit;
}

__device__ inline bool unrealizable(const DevMir VL_GLOBAL &m, uint32_t attr, uint32_t F, uint32_t p) {
  const uint32_t cls = attr_class(attr), width = attr_width(attr), align = attr_align(attr);
  bool bad = p + width > F;
  bad |= (align & (align - 1)) ? (p % align != 0) : ((p & (align - 1)) != 0);
  if (m.has_reserved) {
    for (uint32_t r = p; r < p + width; ++r)
      if (r < 512 && ((m.reserved[cls][r >> 5] >> (r & 31)) & 1u)) bad = true;
  }
  return bad;
}

// Turns the winning key of a candidate row (one per lane) into its result record.  Safety results get their pair from k_resolve.
__device__ inline void finish_row(const DevJob &J, uint32_t k, uint32_t key) {
  const DevMir VL_GLOBAL &m = *as_global(J.mir);
  const DevLive VL_GLOBAL &L = *as_global(J.live);
  vl_result r = {VL_STATUS_OK, 0, 0, 0};
  if (key != kKeyOk) {
    const uint32_t pos = key & kKeyPos;
    switch (key >> 28) {
      case 0: {
        const uint32_t v = m.occ_vreg[pos];
        r = {VL_STATUS_CONSISTENCY, pos, v, L.first[v]};
        if (m.occ_src) r = {VL_STATUS_CONSISTENCY, m.occ_src[pos], m.val_vreg[v], m.occ_src[L.first[v]]};   // in the caller's numbering
        break;
      }
      case 1: {
        const uint32_t v = m.occ_vreg[pos];
        r = {VL_STATUS_REALIZABILITY, pos, v, bad_bits(m, m.vattr[v], cand_at(J, k, pos))};
        if (m.occ_src) { r.where = m.occ_src[pos]; r.a = m.val_vreg[v]; }
        break;
      }
      default: r = {VL_STATUS_SAFETY, pos, kNone, kNone}; break;
    }
  }
  J.out[k] = r;
}

// kOne: the call has one job, which comes as a kernel argument (no table to upload, and a level of
// dependent reads less at the start of every workgroup).
template <uint32_t kRingStride, bool kT, bool kDirect, bool kOne>
__global__ __launch_bounds__(kWalkThreads) __attribute__((amdgpu_waves_per_eu(kT || kDirect ? 6 : 5))) void k_walk(const DevJob one, const DevJob *__restrict__ jobs, uint32_t n_jobs, const Board board) {
  // Workgroups go to the eight dies of the device in turn, each die with an L2 of its own.
  // Inside every 16 consecutive workgroup indices, units 2x and 2x + 1 are given to indices
  // x and x + 8: the two candidate groups of one tile (neighbouring units when a job has two
  // groups) then run on the same die and read the tile's stream records through one L2.
  uint32_t unit = blockIdx.x;
  if ((unit | 15u) < gridDim.x) unit = (unit & ~15u) | ((unit & 7u) << 1) | ((unit >> 3) & 1u);
  const uint32_t job = kOne ? 0u : find_job(jobs, n_jobs, unit, &DevJob::unit_base);
  const DevJob J = kOne ? one : jobs[job];
  const DevMir VL_GLOBAL &m = *as_global(J.mir);
  const DevLive VL_GLOBAL &L = *as_global(J.live);
  // arrays of the kernel and of its analysis, as global pointers
  const auto g_occ_off = m.occ_off, g_occ_instr = m.occ_instr;
  const auto g_prev_occ = L.prev_occ, g_evt_cut = L.evt_cut;
  const auto g_seed_off = L.seed_off, g_tile_range = L.tile_range;
  const u32x4 VL_GLOBAL *g_chk = L.chk, *g_seeds = L.seeds;
  const u32x4 VL_GLOBAL *g_plan = L.plan;
  const uint32_t local = unit - J.unit_base;
  // this workgroup's tile: J.span neighbouring tiles of the analysis, walked as one (the events of a
  // range of tiles follow each other, and what is live into the first starts it)
  const uint32_t tile = local / J.n_groups * J.span, group = local % J.n_groups;
  const uint32_t row0 = group * J.rows;
  Walk w;
  w.tid = threadIdx.x;
  w.lane = threadIdx.x & 63u;
  // the occupancy role moves from wavefront to wavefront with the workgroup index, so
  // that neighbouring workgroups do not all put it on the same SIMD
  const uint32_t role = __builtin_amdgcn_readfirstlane(((threadIdx.x >> 6) + blockIdx.x) % (1u + kCheckWaves));
  w.nrows = group + 1 == J.n_groups ? J.K - row0 : J.rows;   // the last group takes what is left
  const bool active = w.lane < w.nrows;
  w.row = active ? w.lane : 0u;
  w.rows = as_global(J.cand) + (kT ? (uint64_t)row0 : (uint64_t)row0 * J.ld);
  w.ld = J.ld;
  w.n_occ = m.O;
  w.keys = m.occ_words * 64;
  const uint32_t evb = (w.keys + 64) * 4;   // byte offset of the occupancy wavefront's event buffer: 64 records of 16 bytes
  w.ring16 = (w.keys + 64 + 256) * 2;
  for (uint32_t x = w.tid; x < m.occ_words * 64; x += kWalkThreads) vl_lds[x] = 0;
  if (w.tid < 64) vl_lds[w.keys + w.tid] = kKeyOk;
  if (!kT) {
    // ring entries of the rows past the group's last: zero, and never written again
    const uint32_t spare = kRingStride - w.nrows;
    for (uint32_t x = w.tid; x < spare * kRing; x += kWalkThreads) VL_LDS16[w.ring16 + (x / spare) * kRingStride + w.nrows + x % spare] = 0;
  }
  // per-class file size and first mask word, one class per lane, read back by lane index
  const uint32_t cls_tab_v = w.lane < m.C ? ((uint32_t)m.class_size[w.lane] | ((uint32_t)m.class_word[w.lane] << 16)) : 0u;
  uint32_t key = kKeyOk;   // event role and far checks: this lane's row

  const uint32_t i0 = tile * L.tile_len, i1 = min(m.N, i0 + J.span * L.tile_len);
  const uint32_t oa = g_occ_off[i0], ob = g_occ_off[i1];      // the tile's occurrences
  const uint32_t ea = g_tile_range[2 * tile], eb = g_tile_range[2 * min(tile + J.span, L.T) - 1];   // its events
  const uint32_t ca = oa / kChunk;
  const uint32_t c_end = ob > oa ? (ob - 1) / kChunk + 1 : ca;   // chunks [ca, c_end)
  // the ring starts one chunk before the tile's first occurrence, so that nearby history is in LDS
  const uint32_t c_first = ca > 0 ? ca - 1 : 0;
  w.lo = c_first * kChunk;
  w.hi = w.lo;      // nothing readable yet
  __syncthreads();  // masks and keys are cleared

  // ---- occupancy events (lane = candidate) ----
  // Events are replayed in instruction order, so the first clash of a row is the one to
  // report; after it the row's mask is no longer exact and its later clashes are ignored.
  // (The key names the occurrence until the wavefront is done; its instruction is read once, for
  // all rows together.  Reading it at each clash cost a trip to memory per clash.)
  uint32_t alive = 0xFFFFFFFFu;
  auto clash = [&](uint32_t hit, uint32_t o) __attribute__((always_inline)) {
    if (hit & alive) { key = kKeySafe | o; alive = 0; }
  };
  // flips the range of a tuple whose base register is p (any shape of tuple)
  auto apply1 = [&](uint32_t o, uint32_t attr, bool tested, uint32_t p) __attribute__((always_inline)) {
    const Touch t = locate(w, attr, __builtin_amdgcn_readlane(cls_tab_v, attr_class(attr)), p);
    const uint32_t hit = flip(t, attr_straddle(attr));
    if (tested) clash(hit, o);
  };
  const uint32_t my_ring = (w.ring16 + w.row) * 2u;   // byte offset of this lane's row in ring slot 0
  const uint32_t my_occ = w.lane * 4;                 // byte offset of this lane's column of mask words
  char *const lds_bytes = reinterpret_cast<char *>(vl_lds);
  // (nothing is computed from the records here: they are for the next chunk, and the computation
  // would wait for them in this one; with the waits that reads_done keeps off the usual path, 256
  // programs x 100 samples: a step of 800 us instead of 788, 64 large programs 316 instead of 304)
  auto fetch_records = [&](uint32_t from, uint32_t to) __attribute__((always_inline)) {
    u32x4 r = 0;
    if (from + w.lane < to) r = g_plan[from + w.lane];
    return r;
  };
  // Replays a batch of up to 64 records held one per lane (lanes past the batch hold zero
  // records, which flip nothing).
  constexpr int G = 8;
  auto replay = [&](u32x4 r, uint32_t cnt) __attribute__((always_inline)) {
    r.x = (r.x & 0xFFu) * (kRingStride * 2u);   // byte offset of the ring slot (the vreg above it is for the kernels that rebuild P(i))
    if (__any((r.w & kEvtSlow) != 0)) {
      // rare: a tuple that may cross a mask word, or a register from outside the ring
      for (uint32_t j = 0; j < cnt; ++j) {
        const uint32_t sw = __builtin_amdgcn_readlane(r.w, j), o = sw & 0xFFFFFFu;
        const bool slow = (sw & kEvtSlow) != 0;
        const uint32_t attr = slow ? g_chk[o].y >> 16 : 0u;
        const uint32_t p = slow ? fetch<kRingStride, kT>(w, o) : *reinterpret_cast<const uint16_t *>(lds_bytes + my_ring + __builtin_amdgcn_readlane(r.x, j));
        if (slow) {
          apply1(o, attr, (sw & kEvtTested) != 0, p);
        } else {
          const uint32_t msk = (uint32_t)__builtin_amdgcn_readlane(r.y, j) << (p & 31u);
          const uint32_t old = __hip_atomic_fetch_xor(
              reinterpret_cast<uint32_t *>(lds_bytes + ((((p >> 5) & 15u) << 8) + my_occ + __builtin_amdgcn_readlane(r.z, j))), msk,
              __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
          if (sw & kEvtTested) clash(old & msk, o);
        }
      }
      reads_done();
      return;
    }
    typedef __attribute__((address_space(3))) u32x4 lds_u32x4;
    typedef __attribute__((address_space(3))) uint16_t lds_u16;
    typedef __attribute__((address_space(3))) uint32_t lds_u32;
    // LDS addresses as integers with the array's own address folded in once
    const uint32_t lds0 = (uint32_t)(size_t)(lds_u32 *)vl_lds;
    const uint32_t a_ev = lds0 + evb, a_ring = lds0 + my_ring, a_occ = lds0 + my_occ;
    // The batch goes through LDS: every lane writes its record in the form the replay uses
    // (x: byte offset of the carrying occurrence's ring slot, y: the tuple's mask at bit 0,
    // z: byte offset of the class's first mask word, w: all ones for an occupy that is
    // tested), and event j is then read back by all lanes at once from one address, so that
    // its fields arrive in vector registers without lane reads or scalar traffic.
    {
      u32x4 t = r;
      t.w = (uint32_t)((int32_t)r.w >> 31);
      *(lds_u32x4 *)(size_t)(a_ev + w.lane * 16u) = t;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    // Eight events per turn of the loop: their records, their registers, their mask updates
    // and their tests are each issued back to back.  (What bounds this wavefront is the number
    // of instructions it has to issue, not the LDS round trips: keeping a second group in
    // flight, or a four-stage software pipeline over groups of four, made it no faster.)
    constexpr int H = 8;
    struct Ev { uint32_t y, zb, t, p; };
    auto fetch_group = [&](uint32_t g0, Ev (&e)[H]) __attribute__((always_inline)) {
      u32x4 x[H];
      uint32_t a_group = a_ev + g0 * 16u;
      asm volatile("" : "+v"(a_group));   // the reads differ by constant offsets from it, not by an addition each
#pragma unroll
      for (int t = 0; t < H; ++t) x[t] = *(lds_u32x4 *)(size_t)(a_group + t * 16u);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int t = 0; t < H; ++t) {
        e[t].y = x[t].y; e[t].zb = x[t].z; e[t].t = x[t].w;
        e[t].p = *(lds_u16 *)(size_t)(a_ring + x[t].x);
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    auto apply_group = [&](uint32_t g0, Ev (&e)[H], uint32_t (&hit)[H]) __attribute__((always_inline)) {
#pragma unroll
      for (int t = 0; t < H; ++t) {
        e[t].y <<= e[t].p & 31u;
        e[t].p = __hip_atomic_fetch_xor((lds_u32 *)(size_t)(((e[t].p << 3) & 0xF00u) + e[t].zb + a_occ), e[t].y,
                                        __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int t = 0; t < H; ++t) hit[t] = e[t].p & e[t].y & e[t].t;
    };
    auto settle = [&](uint32_t g0, uint32_t (&hit)[H]) __attribute__((always_inline)) {
      uint32_t any_hit = 0;
#pragma unroll
      for (int t = 0; t < H; ++t) any_hit |= hit[t];
      if (__any((any_hit & alive) != 0)) {
#pragma unroll
        for (int t = 0; t < H; ++t) clash(hit[t], __builtin_amdgcn_readlane(r.w, g0 + t) & 0xFFFFFFu);
      }
    };
    for (uint32_t g0 = 0; g0 < cnt; g0 += H) {
      Ev e_[H];
      uint32_t h_[H];
      fetch_group(g0, e_);
      apply_group(g0, e_, h_);
      settle(g0, h_);
    }
    __builtin_amdgcn_wave_barrier();   // the buffer is rewritten by the next batch
  };
  // events [from, to); `first` holds the records [from, from + 64) fetched ahead
  auto events = [&](uint32_t from, uint32_t to, u32x4 first) __attribute__((always_inline)) {
    for (uint32_t e = from; e < to; e += 64) {
      u32x4 r = first;
      if (e != from) {
        r = fetch_records(e, to);
        reads_done();
      }
      if (e + w.lane >= to) r = 0;
      replay(r, min(64u, to - e));
    }
  };
  // Register cache of a check wavefront, for consistency links that reach back beyond the
  // ring: slot s holds, one candidate per lane (16 bits, two slots per register), the
  // registers of the occurrence named by lane s of cache_tag.  Slots are filled in turn (the
  // oldest entry goes) and found by comparing all tags at once; a miss only means that the
  // value is gathered from memory instead.
  constexpr uint32_t kCacheSlots = 32;   // two per register
  typedef uint32_t cache_t __attribute__((ext_vector_type(kCacheSlots / 2)));   // a vector, so that it stays in registers
  cache_t cache = 0;
  uint32_t cache_tag = kNone, cache_next = 0;
  auto cache_put = [&](uint32_t o, uint32_t val) __attribute__((always_inline)) {
    const uint32_t slot = cache_next;
    cache_next = (cache_next + 1u) % kCacheSlots;
    const uint32_t both = cache[slot >> 1];
    cache[slot >> 1] = (slot & 1u) ? ((both & 0xFFFFu) | (val << 16)) : ((both & 0xFFFF0000u) | val);
    if (w.lane == slot) cache_tag = o;
  };

  // The values live into the tile: their registers mostly lie before the ring and are
  // gathered from memory, eight gathers in flight.  Every entry flips its own bits, in any
  // order, before the first barrier: the three check wavefronts share the list by the owner
  // of the source occurrence (index modulo three), one candidate per lane, and keep the
  // registers of the values whose first mention in the tile they will check (kSeedLinked),
  // so that such a link is not gathered a second time long after the line has left the caches.
  auto seed_events = [&](uint32_t from, uint32_t to, uint32_t part) __attribute__((always_inline)) {
    for (uint32_t base = from; base < to; base += 64) {
      const uint32_t cnt = min(64u, to - base);
      u32x4 r = 0;
      if (w.lane < cnt) r = g_seeds[base + w.lane];
      const bool any_slow = __any((r.w & kEvtSlow) != 0);
      uint64_t mine = __ballot(w.lane < cnt && (r.w & 0xFFFFFFu) % kCheckWaves == part);
      while (mine) {
        uint32_t idx[G], p[G];
#pragma unroll
        for (int t = 0; t < G; ++t) {
          idx[t] = mine ? (uint32_t)__builtin_ctzll(mine) : 64u;   // 64: no entry
          mine &= mine - 1;   // (zero stays zero)
        }
#pragma unroll
        for (int t = 0; t < G; ++t)
          p[t] = from_memory<kT>(w, __builtin_amdgcn_readlane(r.w, idx[t] & 63u) & 0xFFFFFFu);
#pragma unroll
        for (int t = 0; t < G; ++t) {
          if (idx[t] == 64u) continue;
          const uint32_t sw = __builtin_amdgcn_readlane(r.w, idx[t]), o = sw & 0xFFFFFFu;
          if (any_slow) {
            apply1(o, g_chk[o].y >> 16, false, p[t]);
          } else {
            const uint32_t msk = (uint32_t)__builtin_amdgcn_readlane(r.y, idx[t]) << (p[t] & 31u);
            __hip_atomic_fetch_xor(reinterpret_cast<uint32_t *>(lds_bytes + ((((p[t] >> 5) & 15u) << 8) + my_occ +
                                                                               __builtin_amdgcn_readlane(r.z, idx[t]))),
                                   msk, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
          }
          if (sw & kSeedLinked) cache_put(o, p[t]);
        }
      }
    }
  };

  // ---- checks of one chunk (lane = check, loop over rows) ----
  // Per lane: ring offsets of the occurrence and of the previous occurrence of its vreg,
  // and for a first occurrence the alignment mask and the largest base that fits.  Per row:
  // two reads and three compares, identical for every lane.
  auto load_chk = [&](uint32_t c) __attribute__((always_inline)) {
    const uint32_t o = c * kChunk + w.lane;
    u32x4 r = nothing_to_check(c, w.lane);
    if (o >= oa && o < ob) r = g_chk[o];
    return r;
  };
  auto checks = [&](uint32_t c, uint32_t part, const u32x4 rec) __attribute__((always_inline)) {
    const uint32_t o = c * kChunk + w.lane;
    const uint32_t fl = rec.x & 0xFFu, attr = rec.y >> 16, delta = rec.y & 0xFFFFu;
    const bool is_chk = (fl & kPlanChk) != 0;
    const uint32_t prev = o - delta;
    const bool near = (fl & kChkNear) && prev >= w.lo;   // the ring starts at the tile's first staged chunk
    const bool far = is_chk && !near;
    const bool generic = (fl & kChkGeneric) != 0;
    // Four rows per 8-byte read, two rows per 32-bit operation.  What is wrong in a row
    // leaves a non-zero half-word: p ^ q (differs from the previous occurrence),
    // p & (align - 1), and p ^ min(p, limit) (beyond the last base that fits).  Rows past
    // the last candidate hold zeros.  The rows are first taken together: differences and
    // registers are or'ed and the largest register kept, three operations for two rows, since
    // instructions are what the kernel is short of (each row's own test takes five).  Only when
    // something is non-zero are the rows looked at one by one.
    typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
    const uint32_t amask2 = rec.z, limit2 = rec.w;
    constexpr uint32_t slot8 = kRingStride / 4;   // a ring slot in 8-byte units
    const uint32_t a_p = (w.ring16 >> 2) + ((rec.x >> 8) & 0xFFFu) * slot8;          // in 8-byte units
    const uint32_t a_q = near ? (w.ring16 >> 2) + (rec.x >> 20) * slot8 : a_p;
    const uint64_t *lds64 = reinterpret_cast<const uint64_t *>(vl_lds);
    auto wrong2 = [&](uint32_t pp, uint32_t qq) __attribute__((always_inline)) {
      const u16x2 mn = __builtin_elementwise_min(__builtin_bit_cast(u16x2, pp), __builtin_bit_cast(u16x2, limit2));
      return (pp ^ qq) | (pp & amask2) | (pp ^ __builtin_bit_cast(uint32_t, mn));
    };
    uint32_t differ = 0, bits = 0;
    u16x2 top = 0;
    auto take = [&](uint64_t p4, uint64_t q4) __attribute__((always_inline)) {
      const uint32_t p0 = (uint32_t)p4, p1 = (uint32_t)(p4 >> 32);
      differ = __builtin_amdgcn_bitop3_b32(p0, (uint32_t)q4, differ, 0xBE);   // (a ^ b) | c, which the compiler takes apart
      differ = __builtin_amdgcn_bitop3_b32(p1, (uint32_t)(q4 >> 32), differ, 0xBE);
      bits |= p0 | p1;
      top = __builtin_elementwise_max(top, __builtin_bit_cast(u16x2, p0));
      top = __builtin_elementwise_max(top, __builtin_bit_cast(u16x2, p1));
    };
    // this wavefront's third of the row quads, two quads (a 16-byte read on either side) at a time
    // (four at a time cost the row-major variants registers they don't have: 403 us instead of 357 for 25,600 samples)
    const uint32_t n_quad = (w.nrows + 3) / 4;
    const uint32_t q_lo = part * n_quad / kCheckWaves, q_hi = (part + 1) * n_quad / kCheckWaves;
    uint32_t qd = q_lo;
    auto take_quads = [&](auto n) __attribute__((always_inline)) {
      constexpr uint32_t N = decltype(n)::value;
      uint64_t pv[N], qv[N];
#pragma unroll
      for (uint32_t t = 0; t < N; ++t) { pv[t] = lds64[a_p + qd + t]; qv[t] = lds64[a_q + qd + t]; }
#pragma unroll
      for (uint32_t t = 0; t < N; ++t) take(pv[t], qv[t]);
      qd += N;
    };
    while (qd + 2 <= q_hi) take_quads(std::integral_constant<uint32_t, 2>{});
    if (qd < q_hi) take_quads(std::integral_constant<uint32_t, 1>{});
    const uint32_t acc = differ | (bits & amask2) |
                         (__builtin_bit_cast(uint32_t, top) ^ __builtin_bit_cast(uint32_t, __builtin_elementwise_min(top, __builtin_bit_cast(u16x2, limit2))));
    if (__any(acc != 0 || generic)) {
      // rare: attribute row by row.  A row's smallest failing key is its first failing
      // consistency check, else its first failing first mention: bits of two lane masks, kept in
      // the lane that stands for the row.  (A reduction over the wavefront for every failing row, and
      // the reads at clashes, were what a chunk with failures waited for: verification of 200
      // instructions with half of 64 samples damaged 33.3 us, 26.0 without them.)
      const uint64_t links = __ballot(is_chk);
      for (uint32_t qd = q_lo; qd < q_hi; ++qd) {
        const uint64_t pv = lds64[a_p + qd], qv = lds64[a_q + qd];
        const uint32_t wrong[2] = {wrong2((uint32_t)pv, (uint32_t)qv), wrong2((uint32_t)(pv >> 32), (uint32_t)(qv >> 32))};
        if (!__any((wrong[0] | wrong[1]) != 0 || generic)) continue;
#pragma unroll
        for (uint32_t t = 0; t < 4; ++t) {
          const uint32_t r = 4 * qd + t;
          bool bad = ((wrong[t >> 1] >> (16u * (t & 1u))) & 0xFFFFu) != 0;
          if (generic && r < w.nrows) bad = unrealizable(m, attr, m.class_size[attr_class(attr)], (uint32_t)(pv >> (16u * t)) & 0xFFFFu);
          const uint64_t fails = __ballot(bad), broken = fails & links;
          if (fails) {
            const uint32_t k = (broken ? kKeyCons | (uint32_t)__builtin_ctzll(broken) : kKeyReal | (uint32_t)__builtin_ctzll(fails)) + c * kChunk;
            if (w.lane == r) key = min(key, k);
          }
        }
      }
    }
    // Links that reach back beyond the ring, one candidate per lane.  The earlier value is
    // taken from the wavefront's register cache when its tag still names that occurrence,
    // otherwise from memory.  A link belongs to the wavefront that owns its earlier
    // occurrence (index modulo three), which is also the one that cached it.
    const bool sat = delta == 0xFFFFu;
    uint64_t todo = __ballot(far && (sat ? w.lane % kCheckWaves == part : prev % kCheckWaves == part));
    while (todo) {
      const uint32_t j = __builtin_ctzll(todo);
      todo &= todo - 1;
      const uint32_t oj = c * kChunk + j;
      const uint32_t dj = __builtin_amdgcn_readlane(delta, j);
      const uint32_t pv = VL_LDS16[w.ring16 + (oj % kRing) * kRingStride + w.row];
      uint32_t qv;
      if (dj != 0xFFFFu) {
        const uint32_t pj = oj - dj;
        const uint64_t at = __ballot(cache_tag == pj);
        if (at) {
          const uint32_t slot = __builtin_ctzll(at);
          qv = (cache[slot >> 1] >> (16u * (slot & 1u))) & 0xFFFFu;
        } else {
          qv = from_memory<kT>(w, pj);
          reads_done();
        }
      } else {
        qv = from_memory<kT>(w, g_prev_occ[oj]);
        reads_done();
      }
      if (pv != qv) key = min(key, kKeyCons | oj);
    }
    // occurrences whose successor is likely out of reach: keep their registers
    uint64_t keep = __ballot((fl & kPlanKeep) && o % kCheckWaves == part);
    while (keep) {
      const uint32_t j = __builtin_ctzll(keep);
      keep &= keep - 1;
      const uint32_t oj = c * kChunk + j;
      cache_put(oj, VL_LDS16[w.ring16 + (oj % kRing) * kRingStride + w.row]);
    }
  };

  // Schedule.  The three check wavefronts do the staging: while chunk c is processed they
  // write chunk c + 1 over the slots of chunk c - 2 (nobody reads further back than chunk
  // c - 1 any more: kWalkReach) and fetch chunk c + 2.  The occupancy wavefront only replays
  // events: first the tile's live-in values, while the others fill the ring, then per chunk
  // what that chunk releases.  One barrier per chunk; both kinds of wavefront pass the same
  // number of barriers (a tile without operands still replays its events once).
  const uint32_t c_stop = c_end > ca ? c_end : ca + 1;
  // occupancy wavefront: limits of the current chunk's batch, clamped to the tile, and the
  // next chunk's records.  The limits are read with vector loads (the lane-dependent index
  // keeps them off the scalar unit, whose loads would share a counter with the LDS reads).
  const uint32_t n_chunk = (w.n_occ + kChunk - 1) / kChunk;
  uint32_t lane_zero;   // zero in a vector register the compiler cannot see through
  asm volatile("v_mov_b32 %0, 0" : "=v"(lane_zero));
  auto clamp_cut = [&](uint32_t e) __attribute__((always_inline)) { return min(eb, max(ea, e)); };
  if (role == 0) {
    // the occupancy wavefront has the longest chain of dependent steps per chunk: it goes
    // first when it competes for issue with the check wavefronts of other workgroups
    __builtin_amdgcn_s_setprio(3);
    uint32_t cut_lo = ea;
    uint32_t v_cut_next = g_evt_cut[min(ca + 1, n_chunk) + lane_zero];
    u32x4 rec_next = fetch_records(ea, eb);   // the first batch, in flight during the seeds
    __syncthreads();   // chunks up to ca are in the ring
    for (uint32_t c = ca; c != c_stop; ++c) {
      if (c < c_end) w.hi = (c + 1) * kChunk;
      const uint32_t cut_hi = clamp_cut(__builtin_amdgcn_readfirstlane(v_cut_next));
      const uint32_t from = cut_lo, to = c + 1 >= c_end ? eb : cut_hi;
      const u32x4 first = rec_next;
      // fetch ahead for the next chunk, without waiting: its upper limit and the 64 records
      // from its lower limit on (those past its upper limit are dropped before the replay)
      cut_lo = cut_hi;
      v_cut_next = g_evt_cut[min(c + 2, n_chunk) + lane_zero];
      rec_next = fetch_records(cut_lo, eb);
      events(from, to, first);
      __syncthreads();
    }
    if (key != kKeyOk) key = kKeySafe | g_occ_instr[key & kKeyPos];
  } else {
    const uint32_t j = role - 1;
    // row-major staging: this lane's row of every pass, from the word the group's rows begin in
    const uint32_t in_word = (uint32_t)(uintptr_t)w.rows & 2u;
    const __amdgpu_buffer_rsrc_t rows_desc = __builtin_amdgcn_make_buffer_rsrc((void *)((uintptr_t)w.rows - in_word), 0, -1, 0x00020000);
    w.last_piece = (int32_t)((w.n_occ - 1u) / 8u * 16u) - (int32_t)(w.lane & 7u) * 16;
    const bool shifted = !kDirect && (in_word || (w.ld & 1u));   // some rows begin in the middle of a word
#pragma unroll
    for (int h = 0; h < kStagePasses; ++h) {
      const uint32_t q = j + kCheckWaves * h, r = staged_row(w.lane, q);
      const bool has_row = !kT && q < 8u && r < w.nrows;
      const uint32_t from = (uint32_t)((r * w.ld + (w.lane & 7u) * 8u) * 2u) + in_word;
      w.from_row[h] = has_row ? (kDirect ? from : (from & ~3u) | ((from >> 1) & 1u)) : kNone;
      if (!kT && !kDirect) w.pre[h][4] = 0;
      w.to_ring[h] = w.ring16 + (w.lane & 7u) * 8u * kRingStride + r;
    }
    auto stage_load = [&](uint32_t c0) __attribute__((always_inline)) {
      if (kDirect) load_chunk_direct(w, c0, rows_desc);
      else if (kT) load_chunk_occ(w, c0, j);
      else load_chunk_ragged(w, c0, rows_desc, shifted);
    };
    auto stage_store = [&](uint32_t c0) __attribute__((always_inline)) {
      if (kDirect) store_chunk_direct<kRingStride>(w, c0);
      else if (kT) store_chunk_occ<kRingStride>(w, c0, j);
      else store_chunk_ragged<kRingStride>(w, c0);
    };
    for (uint32_t c = c_first; c <= ca && c < c_end; ++c) {   // history chunk and the tile's first chunk
      stage_load(c * kChunk);
      stage_store(c * kChunk);
    }
    if (ca + 1 < c_end) stage_load((ca + 1) * kChunk);
    u32x4 chk_next = load_chk(ca);
    if (tile > 0) seed_events(g_seed_off[tile], g_seed_off[tile + 1], j);   // this wavefront's share of the live-in list
    __syncthreads();
    for (uint32_t c = ca; c != c_stop; ++c) {
      if (c < c_end) {
        if (c + 1 < c_end) {
          stage_store((c + 1) * kChunk);
          if (c + 2 < c_end) stage_load((c + 2) * kChunk);
        }
        w.hi = (c + 1) * kChunk;
        const u32x4 raw = chk_next;
        chk_next = load_chk(c + 1);   // in flight while this chunk is checked
        checks(c, j, raw);
      }
      __syncthreads();
    }
  }
  __syncthreads();
  if (active && key != kKeyOk) atomicMin(&vl_lds[w.keys + w.lane], key);
  __syncthreads();
  // The tile reports to the group's board; the tile that reports last turns the group's keys into
  // results (one wavefront, a row per lane).  Keys and counter are only touched by atomics, which
  // the dies of the device see in one order; the returned values keep a wavefront's own in order.
  if (w.tid >= 64) return;
  uint32_t found = w.tid < w.nrows ? vl_lds[w.keys + w.tid] : kKeyOk;
  // (the job's entry is read again rather than kept in scalar registers through the walk, which
  // has none to spare; `one` is the first kernel argument)
  const DevJob VL_CONSTANT *entry = kOne ? (const DevJob VL_CONSTANT *)__builtin_amdgcn_kernarg_segment_ptr() : (const DevJob VL_CONSTANT *)(uintptr_t)jobs;
  asm volatile("" : "+s"(entry));
  const DevJob E = *((const DevJob *)entry + job);
  const uint32_t T = E.n_spans, row = (unit - E.unit_base) % E.n_groups * E.rows + w.tid;
  if (T > 1) {
    uint32_t *const my_key = board.keys + E.row_base + row;
    uint32_t before = 0;
    if (found != kKeyOk) before = __hip_atomic_fetch_max(my_key, ~found, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" : "+v"(before) : : "memory");
    uint32_t n_before = 0;
    uint32_t *const counter = board.arrived + E.group_base + (unit - E.unit_base) % E.n_groups;
    if (w.tid == 0) n_before = __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (__builtin_amdgcn_readfirstlane(n_before) + 1u != T) return;
    if (w.tid < w.nrows) found = ~__hip_atomic_exchange(my_key, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (w.tid == 0) __hip_atomic_store(counter, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (w.tid < w.nrows) finish_row(E, row, found);
}

// For a candidate whose first violation is a register clash at instruction i: the
// lexicographically smallest pair (a < b) of one class, both in P(i) = live_after(i) + defs(i),
// with overlapping ranges.  At the first clashing instruction every clashing pair contains a
// vreg that the instruction defines, so only pairs (definition, anything in P(i)) are
// examined.  P(i) is rebuilt as a bitset in LDS the way the walk builds occupancy, but over
// vregs instead of registers (RecordsOfP); a candidate that got this far is consistent, so any occurrence
// of a member has the value's register.
// What bounds it is the chain of reads: result, offsets of i, events of i and its operands, records, registers.
// Short lists are kept as records between the flips and the comparison; of longer ones one word is read of each record, and
// the members are listed from the bitset and looked up a lane each, two trips more.  (Reading the rest of a long list a
// record at a time, before and after the flips: 4,000 instructions in one tile, 50 rows to resolve 21.6 us, 10.2 this way,
// 11.3 with lists for all; 256 programs in tiles of 512, 27.7 and 25.3.  Five events kept instead of three, and the
// registers that takes: 28.8, packed into two words each 25.1, but 4.6 instead of 4.4 for 200 instructions x 64.)
// The workgroups of a group of rows share out the rows that
// failed on safety.  kShared: it leaves the board zero (Board).
constexpr uint32_t kResolveThreads = 128;   // at least kMaxOperands; 64 and 256 were measured slower
constexpr uint32_t kResolveMembers = 512;   // members of P(i) that are listed; with more, every vreg gets a turn
template <bool kOne, bool kShared>
__global__ __launch_bounds__(kResolveThreads) void k_resolve(const DevJob *__restrict__ jobs, uint32_t n_jobs, const DevJob one, uint32_t per_group, uint32_t n_groups,
                                                             const Board board) {
  extern __shared__ uint32_t in_p[];   // [W]
  __shared__ unsigned long long best;
  __shared__ uint32_t dv[kMaxOperands], dp[kMaxOperands], da[kMaxOperands], nd, members[kResolveMembers], n_members;
  const uint32_t global_group = blockIdx.x / per_group, mine_first = blockIdx.x % per_group;
  const DevJob J = kOne ? one : jobs[find_job(jobs, n_jobs, global_group, &DevJob::group_base)];
  const uint32_t group = global_group - J.group_base, row0 = group * J.rows, tid = threadIdx.x;
  const uint32_t nrows = group + 1 == J.n_groups ? J.K - row0 : J.rows, lane = tid & 63u;
  vl_result VL_GLOBAL *const out = as_global_rw(J.out) + row0;
  const DevMir VL_GLOBAL &m = *as_global(J.mir);
  const DevLive VL_GLOBAL &L = *as_global(J.live);
  // this workgroup's share of the group's rows (at most 64) that failed on safety, by rank
  const uint32_t my_row = min(lane, nrows - 1u), status = out[my_row].status, where = out[my_row].where;
  // The board of a group, behind the read above, since reads wait for the stores before them.  One job: by the
  // workgroups that start first, since the launch ends with its last store.  Several: by each group's first.
  // (60 instructions x 8, 64 and 4,000 samples, us per call without / with: 11.2 / 11.4, 15.8 / 16.1, 19.1 / 20.1;
  // 256 programs x 100: 29.2 us for the launch, 33.6 with.)
  if (kShared && (kOne ? blockIdx.x < n_groups : mine_first == 0)) {
    const uint32_t g = kOne ? blockIdx.x : group, n = g + 1 == J.n_groups ? J.K - g * J.rows : J.rows;
    auto clear = [](uint32_t *p) { __hip_atomic_store(p, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
    if (tid < n) clear(board.keys + J.row_base + g * J.rows + tid);
    if (tid == 64) clear(board.arrived + J.group_base + g);
    if (tid == 65 && blockIdx.x == 0) clear(board.arrived - kHeadWords);   // the counter of the stream's reductions
  }
  uint64_t todo = __ballot(lane < nrows && status == VL_STATUS_SAFETY);
  // (the first of this workgroup's rows; where none failed, nothing is counted off: 64 straight-line programs x 64 samples that all
  // verify 22.8 us a call, 26.4 when every workgroup counted up to its rank)
  for (uint32_t x = 0; x < mine_first && todo; ++x) todo &= todo - 1;
  while (todo) {
    const uint32_t row = (uint32_t)__builtin_ctzll(todo), k = row0 + row, i = __builtin_amdgcn_readlane(where, row);
    for (uint32_t x = 0; x < per_group && todo; ++x) todo &= todo - 1;
    if (kShared && i >= m.N) continue;   // (not a result of this call: calls overlapped against the rules)
    const uint32_t o_lo = m.occ_off[i], n_ops = m.occ_off[i + 1] - o_lo;
    const RecordsOfP p = records_of_p(m, L, i);
    for (uint32_t x = tid; x < m.W; x += kResolveThreads) in_p[x] = 0;
    // the vregs the instruction writes and their registers: one operand per lane
    uint32_t my_v = kNone, my_p = 0;
    if (tid < n_ops) {
      const uint32_t flags = m.occ_flags[o_lo + tid], v = m.occ_vreg[o_lo + tid];
      my_p = cand_at(J, k, o_lo + tid);
      if (flags & VL_OCC_DEF) my_v = v;
    }
    KeptRecords<1, 3, kResolveThreads> kept;
    const bool fit = kept.fit(p);
    if (fit) kept.load(L, p, tid);
    if (tid < kMaxOperands) {   // one wavefront
      const uint32_t attr = my_v != kNone ? m.vattr[my_v] : 0u;
      const uint64_t defs = __ballot(my_v != kNone);
      if (my_v != kNone) {
        const uint32_t slot = (uint32_t)__popcll(defs & ((1ull << tid) - 1ull));
        dv[slot] = my_v; dp[slot] = my_p; da[slot] = attr;
      }
      if (tid == 0) { best = ~0ull; nd = (uint32_t)__popcll(defs); n_members = 0; }
    }
    static_assert(kMaxOperands == 64, "a wavefront");
    __syncthreads();
    if (fit) kept.flip(in_p);
    else flip_members_of_p(L, p, in_p, tid, kResolveThreads);
    __syncthreads();
    unsigned long long mine = ~0ull;
    const uint32_t n_defs = nd;
    auto examine = [&](uint32_t x, uint32_t wx, uint32_t cls_word, uint32_t px) {
      for (uint32_t t = 0; t < n_defs; ++t) {
        const uint32_t d = dv[t], ad = da[t];
        if (d == x || attr_word(ad) != cls_word) continue;   // (classes begin at different mask words)
        const uint32_t pd = dp[t], wd = attr_width(ad);
        if (pd < px + wx && px < pd + wd) {
          // (a program with lanes as values reports the caller's vregs: the smallest pair of those)
          const uint32_t a = m.val_vreg ? m.val_vreg[d] : d, b = m.val_vreg ? m.val_vreg[x] : x;
          const unsigned long long pr = ((unsigned long long)min(a, b) << 32) | max(a, b);
          mine = pr < mine ? pr : mine;
        }
      }
    };
    if (fit) {
      uint32_t px[kept.kAll];
#pragma unroll
      for (uint32_t u = 0; u < kept.kAll; ++u) {   // (all in flight)
        u32x4 &r = kept.rec[u];
        px[u] = 0;
        if (r.y && is_member(in_p, r.x >> 8)) px[u] = cand_at(J, k, r.w & 0xFFFFFFu);
        else r.y = 0;
      }
#pragma unroll
      for (uint32_t u = 0; u < kept.kAll; ++u) {
        const u32x4 r = kept.rec[u];
        if (r.y) examine(r.x >> 8, (uint32_t)__popc(r.y), r.z / 256u, px[u]);
      }
    } else {
      auto look_up = [&](uint32_t x) {
        const uint32_t ax = m.vattr[x], o = L.first[x];
        examine(x, attr_width(ax), attr_word(ax), cand_at(J, k, o));
      };
      list_members(in_p, m.W, members, kResolveMembers, &n_members, tid, kResolveThreads);
      __syncthreads();
      if (n_members <= kResolveMembers) {
        for (uint32_t x = tid; x < n_members; x += kResolveThreads) look_up(members[x]);
      } else {
        for (uint32_t x = tid; x < m.V; x += kResolveThreads)
          if (is_member(in_p, x)) look_up(x);
      }
    }
    if (mine != ~0ull) atomicMin(&best, mine);
    __syncthreads();
    if (tid == 0) {
      out[row].a = (uint32_t)(best >> 32);
      out[row].b = (uint32_t)best;
    }
    __syncthreads();   // the shared arrays are reused by the next row
  }
}

// Job tables on the device: per device a few slots, one per stream that has called, so
// that calls alternating between streams neither wait for each other's table nor overwrite
// a table that kernels of the other stream still read.
struct Slot {
  bool used = false;
  hipStream_t stream = nullptr;
  WalkSpace space;
  uint64_t tick = 0;
};
constexpr int kSlots = 4;
constexpr uint64_t kResolveGroups = 4096;   // workgroups that share out the clashes to resolve, about
struct Scratch {
  std::mutex mu;
  Slot slot[kSlots];
  uint64_t clock = 0;
};
Scratch g_scratch[16];

thread_local hipEvent_t g_time_start = nullptr, g_time_stop = nullptr;

}  // namespace

// measurement hook of the benchmark (include/vl_bench.h), not part of the boundary
extern "C" int32_t vl_verify_time_next(void *start, void *stop) {
  g_time_start = (hipEvent_t)start;
  g_time_stop = (hipEvent_t)stop;
  return VL_OK;
}

namespace {
struct Launch {
  DevJob *dev = nullptr;   // the job table on the device; a single job travels as an argument instead
  DevJob one = {};
  Board board = {};
  bool shared = false;     // other calls may find the board in use, against the rules
  uint32_t *finished = nullptr;   // counter of the stream's reductions, zero between calls
  uint64_t total_rows = 0, groups = 0;
  uint32_t most_span = 1;         // of the analyses
  uint32_t units = 0, maxK = 0, max_words = 0, max_w = 1, max_rows = 0;
  bool all_direct = true;   // every job can be staged with 32-bit offsets and without bounds (DevJob::direct)
};

// results_only: for the kernels that read nothing but the jobs' results (cand and ld are neither checked nor used)
inline int32_t check_job(const vl_job &u, bool transposed, bool results_only) {
  if (!u.mir || !u.live || !u.out || (!u.cand && !results_only)) return VL_E_NULL;
  if (u.mir->magic != kMirMagic || u.live->magic != kLiveMagic || u.live->mir != u.mir) return VL_E_ARG;
  if (u.K == 0 || (!results_only && u.ld < (transposed ? u.K : u.mir->h.O))) return VL_E_SHAPE;
  return VL_OK;
}

// Validates one job, lays out its entry of the device job table and adds it to the launch.
// span: analysis tiles taken at once, where the analysis allows it.
int32_t fill_job(const vl_job &u, bool transposed, DevJob &d, Launch &out, uint32_t span) {
  const int32_t rc = check_job(u, transposed, false);
  if (rc != VL_OK) return rc;
  memset(&d, 0, sizeof(d));
  d.mir = u.mir->dev; d.live = u.live->dev; d.cand = u.cand; d.out = u.out; d.ld = u.ld; d.K = u.K;
  const bool aligned = ((uintptr_t)u.cand & 15) == 0 && (u.ld & 7) == 0;
  d.transposed = transposed ? 1u : 0u;
  // every row has room for whole chunks: the pitch covers the last one
  d.direct = (aligned && !transposed && u.ld >= (((uint64_t)u.mir->h.O + kChunk - 1) / kChunk) * kChunk) ? 1u : 0u;
  out.all_direct = out.all_direct && d.direct;
  // groups of up to 64 candidates; every group but the last has d.rows of them.  Row-major groups span
  // less than 4 GB, so that 32-bit offsets reach every register (a row alone needs less than 32 MB of it)
  constexpr uint64_t kReach = ((1ull << 32) - (1ull << 26)) / 2;
  uint32_t most = 64;
  if (!transposed && u.ld > kReach / 64) most = (uint32_t)std::max<uint64_t>(1, kReach / u.ld);
  d.n_groups = (u.K + most - 1) / most;
  d.rows = (u.K + d.n_groups - 1) / d.n_groups;
  if (transposed) {
    // occurrence-major: a group is copied in 16-byte pieces of 8 candidates, so groups
    // start at multiples of 8; rounding the group size down keeps the groups small
    // (100 candidates: 48 + 52) unless the last one then outgrows a wavefront
    if (!aligned) return VL_E_SHAPE;
    uint32_t base = (u.K / d.n_groups) & ~7u;
    if (base == 0 || u.K - (d.n_groups - 1) * base > 64) {
      base = ((u.K + d.n_groups - 1) / d.n_groups + 7u) & ~7u;
      d.n_groups = (u.K + base - 1) / base;
    }
    d.rows = base;
  }
  const uint32_t last = u.K - (d.n_groups - 1) * d.rows;
  d.unit_base = out.units;
  if (out.total_rows + u.K > 0xFFFFFFFFull) return VL_E_SHAPE;   // (the board has an entry per row)
  d.row_base = (uint32_t)out.total_rows;
  d.group_base = (uint32_t)out.groups;
  out.groups += d.n_groups;
  d.span = std::min(span, u.live->span);
  d.n_spans = (u.live->h.T + d.span - 1) / d.span;
  out.most_span = std::max(out.most_span, u.live->span);
  out.units += d.n_groups * d.n_spans;
  out.maxK = std::max(out.maxK, u.K);
  out.total_rows += u.K;
  out.max_rows = std::max(out.max_rows, std::max(d.rows, last));
  out.max_words = std::max(out.max_words, u.mir->h.occ_words);
  out.max_w = std::max(out.max_w, u.mir->h.W);
  return VL_OK;
}

// The jobs of a call.  Short tiles are cut for programs of few instructions, whatever the number of samples, so that
// few samples keep the device busy; once there are some 900 workgroups (it holds 1,280 to 1,536), halving their
// number costs nothing and saves every second tile's set-up and live-in list.  (Tiles of 32, 64 and 128,
// us per call.  4,000 instructions x 1,000 samples, 2,000 / 1,000 / 500 workgroups: 46, 33, 32;
// 2,000 x 1,000, 1,008 / 504 / 252: 29, 26, 30; 2,000 x 4,000, 3,969 / 1,984 / 992: 70, 54, 47;
// 1,000 x 1,000, 512 / 256 / 128: 23, 24, 28; 400 straight x 4,000, 819 / 441 / 252: 23, 24, 30.)
constexpr uint32_t kEnoughUnits = 900;
int32_t fill_jobs(const vl_job *jobs, uint32_t n_jobs, bool transposed, DevJob *tab, Launch &out) {
  for (uint32_t span = 1;; span *= 2) {
    out = Launch();
    for (uint32_t j = 0; j < n_jobs; ++j) {
      const int32_t rc = fill_job(jobs[j], transposed, tab[j], out, span);
      if (rc != VL_OK) return rc;
    }
    if (out.units <= kEnoughUnits || span >= out.most_span) return VL_OK;
  }
}

__global__ void k_clear_board(uint32_t *p, uint64_t n) {
  for (uint64_t x = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; x < n; x += (uint64_t)gridDim.x * blockDim.x) p[x] = 0;
}

// The calling stream's slot, else a free one, else the least recently used one (whose
// earlier kernels may be anywhere: the device is drained before the slot changes hands).
// Called with the device's scratch locked.
int32_t space_of(Scratch &sc, hipStream_t stream, WalkSpace *&out) {
  Slot *found = nullptr;
  for (Slot &c : sc.slot)
    if (c.used && c.stream == stream) found = &c;
  if (!found)
    for (Slot &c : sc.slot)
      if (!c.used && !found) found = &c;
  if (!found) {
    found = &sc.slot[0];
    for (Slot &c : sc.slot)
      if (c.tick < found->tick) found = &c;
    VL_HIP(hipDeviceSynchronize());
    found->space.n_valid = 0;
  }
  // a recorded pass keeps the memory of its stream; threads that each pass their own default stream share one place
  hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
  if (!found->space.recorded) {
    if (hipStreamIsCapturing(stream, &capture) != hipSuccess) (void)hipGetLastError();   // (the null stream, while another is recorded)
    found->space.recorded = capture != hipStreamCaptureStatusNone || stream == hipStreamPerThread;
  }
  found->used = true;
  found->stream = stream;
  found->tick = ++sc.clock;
  out = &found->space;
  return VL_OK;
}

// Validates the jobs, lays out the device job table and makes sure the device copy is
// current (the copy is skipped when the table is the one the space already holds).  The space is the
// caller's for the duration of the call, and its earlier kernels run on `stream` or have ended.
int32_t prepare_jobs(const vl_job *jobs, uint32_t n_jobs, hipStream_t stream, WalkSpace &s, Launch &out, bool transposed = false,
                     bool results_only = false) {
  std::vector<DevJob> tab;
  if (results_only) {
    // the table a verification call on this stream left behind serves, whatever its candidate
    // layout, when it names the same results
    bool same = n_jobs > 1 && s.n_valid == n_jobs && s.board;
    for (uint32_t j = 0; j < n_jobs; ++j) {
      const int32_t rc = check_job(jobs[j], false, true);
      if (rc != VL_OK) return rc;
      same = same && s.host[j].out == jobs[j].out && s.host[j].K == jobs[j].K;
      out.maxK = std::max(out.maxK, jobs[j].K);
    }
    if (same) {
      out.dev = s.dev;
      out.finished = s.board;
      return VL_OK;
    }
    tab.resize(n_jobs);
    for (uint32_t j = 0; j < n_jobs; ++j) { tab[j].out = jobs[j].out; tab[j].K = jobs[j].K; }
  } else {
    tab.resize(n_jobs);
    const int32_t rc = fill_jobs(jobs, n_jobs, transposed, tab.data(), out);
    if (rc != VL_OK) return rc;
  }
  if (!s.board || (!results_only && (s.groups_cap < out.groups || s.rows_cap < out.total_rows))) {
    VL_HIP(hipStreamSynchronize(stream));   // earlier kernels of the stream may still use the old board
    if (s.board) (void)hipFree(s.board);
    s.board = nullptr; s.groups_cap = s.rows_cap = 0;
    // (reductions use the head alone, and count no rows)
    const uint64_t rows = std::max<uint64_t>(65536, out.total_rows + out.total_rows / 2), groups = std::max<uint64_t>(4096, out.groups + out.groups / 2);
    VL_HIP(device_alloc((void **)&s.board, (size_t)(kHeadWords + rows + groups) * 4));
    k_clear_board<<<256, 256, 0, stream>>>(s.board, kHeadWords + rows + groups);
    s.rows_cap = rows; s.groups_cap = groups;
  }
  if (n_jobs == 1) {
    out.one = tab[0];   // goes to the kernels as an argument
  } else {
    if (s.cap < n_jobs) {
      VL_HIP(hipStreamSynchronize(stream));
      if (s.dev) (void)hipFree(s.dev);
      if (s.staged) (void)hipHostFree(s.staged);
      s.dev = nullptr; s.staged = s.host = nullptr; s.cap = 0; s.n_valid = 0;
      uint32_t cap = std::max(256u, n_jobs);
      VL_HIP(device_alloc((void **)&s.dev, (size_t)cap * sizeof(DevJob)));
      VL_HIP(hipHostMalloc((void **)&s.staged, (size_t)cap * kStaged * sizeof(DevJob), hipHostMallocDefault));
      for (uint32_t t = 0; t < kStaged; ++t) {
        if (!s.copied[t]) VL_HIP(hipEventCreateWithFlags(&s.copied[t], hipEventDisableTiming));
        s.in_flight[t] = false;
      }
      s.cap = cap;
    }
    if (s.n_valid != n_jobs || memcmp(s.host, tab.data(), (size_t)n_jobs * sizeof(DevJob)) != 0) {
      s.turn = (s.turn + 1) % kStaged;
      if (s.in_flight[s.turn]) VL_HIP(hipEventSynchronize(s.copied[s.turn]));
      s.host = s.staged + (size_t)s.turn * s.cap;
      s.n_valid = 0;
      memcpy(s.host, tab.data(), (size_t)n_jobs * sizeof(DevJob));
      // kernels of an earlier call that still read the old device table run on this same
      // stream: the copy below is ordered after them
      VL_HIP(hipMemcpyAsync(s.dev, s.host, (size_t)n_jobs * sizeof(DevJob), hipMemcpyHostToDevice, stream));
      VL_HIP(hipEventRecord(s.copied[s.turn], stream));
      s.in_flight[s.turn] = true;
      s.n_valid = n_jobs;
    }
  }
  out.dev = s.dev;
  out.finished = s.board;
  out.board = Board{s.board + kHeadWords, s.board + kHeadWords + s.groups_cap};
  out.shared = s.recorded;
  return VL_OK;
}

// ---- regeneration-loop reductions ----------------------------------------------------
// Per job the histogram of the statuses and the first accepted candidate.  With
// `stats`, the workgroup that finishes last also totals the jobs' summaries (every field is
// written, nothing needs clearing beforehand; `finished` is left zero).  The summaries reach it
// through stores and loads that all dies see (agent scope).
// What bounds it: waiting for the statuses, 16 bytes apart.  A wavefront reads 256 (many samples: 512)
// at a time.  Jobs of up to kFewSamples get a wavefront each, four to a workgroup; with more in some job,
// every job gets a workgroup of sixteen.  (A wavefront and a
// workgroup per job, 64 jobs: 1,000 samples 7.8 and 10.0 us, 2,000 10.4 and 10.0, 4,000 16.6 and 10.1; one
// job of 65,536: 198 and 24, 54 with a workgroup of four that reads 256 at a time.)
constexpr uint32_t kFewSamples = 2048;
template <bool kMany>
__global__ __launch_bounds__(kMany ? 1024 : 256) void k_summarize(const DevJob *__restrict__ jobs, uint32_t n_jobs, const DevJob one, vl_summary *__restrict__ summaries,
                                                   vl_loop_stats *stats, uint32_t *finished) {
  constexpr uint32_t kWaves = kMany ? 16 : 4, kThreads = 64 * kWaves, kAtOnce = kMany ? 8 : 4;
  const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6, j = kMany ? blockIdx.x : blockIdx.x * kWaves + wave;
  __shared__ uint32_t sums[kMany ? 5 : 1];   // (many) histogram, first accepted
  if (kMany) {
    if (threadIdx.x < 5) sums[threadIdx.x] = threadIdx.x < 4 ? 0u : kNone;
    __syncthreads();
  }
  if (j < n_jobs) {
    const DevJob J = n_jobs == 1 ? one : jobs[j];
    uint32_t hist[4] = {0, 0, 0, 0}, first = kNone;
    // (64 bits: the last step may pass 2^32)
    for (uint64_t k0 = kMany ? wave * 64u * kAtOnce : 0u; k0 < J.K; k0 += 64u * kAtOnce * (kMany ? kWaves : 1u)) {
      uint32_t st[kAtOnce];
#pragma unroll
      for (uint32_t u = 0; u < kAtOnce; ++u) {
        const uint64_t k = k0 + u * 64u + lane;
        st[u] = k < J.K ? J.out[k].status & 3u : 4u;
      }
#pragma unroll
      for (uint32_t u = 0; u < kAtOnce; ++u)
#pragma unroll
        for (uint32_t t = 0; t < 4; ++t) {
          const uint64_t with = __ballot(st[u] == t);
          hist[t] += (uint32_t)__popcll(with);
          if (t == VL_STATUS_OK && with && first == kNone) first = (uint32_t)k0 + u * 64u + (uint32_t)__builtin_ctzll(with);
        }
    }
    if (kMany) {
      if (lane < 4) atomicAdd(&sums[lane], lane == 0 ? hist[0] : lane == 1 ? hist[1] : lane == 2 ? hist[2] : hist[3]);
      if (lane == 4) atomicMin(&sums[4], first);
      __syncthreads();   // (a whole workgroup has the same job)
#pragma unroll
      for (uint32_t t = 0; t < 4; ++t) hist[t] = sums[t];
      first = sums[4];
    }
    first = min(first, J.K);
    const uint32_t word = lane == 0 ? first : lane == 1 ? (first < J.K ? 1u : 0u) : lane == 2 ? hist[0] : lane == 3 ? hist[1] : lane == 4 ? hist[2] : hist[3];
    static_assert(sizeof(vl_summary) == 24, "six words");
    if (lane < 6 && (!kMany || wave == 0)) __hip_atomic_store((uint32_t *)(summaries + j) + lane, word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (!stats) return;
  asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
  __shared__ uint32_t last;
  __shared__ unsigned long long part[kWaves][7];   // per wavefront: passed, most tries, sum of tries, histogram
  __syncthreads();
  if (threadIdx.x == 0) last = __hip_atomic_fetch_add(finished, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u == gridDim.x;
  __syncthreads();
  if (!last) return;
  unsigned long long mine[7] = {0, 0, 0, 0, 0, 0, 0};
  for (uint32_t x = threadIdx.x; x < n_jobs; x += kThreads) {
    uint32_t f[6];
#pragma unroll
    for (uint32_t t = 0; t < 6; ++t) f[t] = __hip_atomic_load((uint32_t *)(summaries + x) + t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const uint32_t tries = f[1] ? f[0] + 1u : n_jobs == 1 ? one.K : jobs[x].K;
    mine[0] += f[1];
    mine[1] = max(mine[1], (unsigned long long)tries);
    mine[2] += tries;
    for (uint32_t t = 0; t < 4; ++t) mine[3 + t] += f[2 + t];
  }
  for (int d = 32; d >= 1; d >>= 1)
#pragma unroll
    for (uint32_t t = 0; t < 7; ++t) {
      const unsigned long long y = __shfl_xor(mine[t], d, 64);
      mine[t] = t == 1 ? max(mine[t], y) : mine[t] + y;
    }
  if (lane == 0)
    for (uint32_t t = 0; t < 7; ++t) part[wave][t] = mine[t];
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long s[7];
    for (uint32_t t = 0; t < 7; ++t) {
      s[t] = part[0][t];
      for (uint32_t k = 1; k < kWaves; ++k) s[t] = t == 1 ? max(s[t], part[k][t]) : s[t] + part[k][t];
    }
    *stats = vl_loop_stats{(uint32_t)s[0], (uint32_t)s[1], s[2], {s[3], s[4], s[5], s[6]}};
    __hip_atomic_store(finished, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}
}  // namespace

extern "C" int32_t vl_summarize_multi(const vl_job *jobs, uint32_t n_jobs, vl_summary *summaries, vl_loop_stats *stats,
                                      vl_stream stream_) {
  if (!jobs || !summaries) return VL_E_NULL;
  if (n_jobs == 0 || n_jobs > 65535) return VL_E_SHAPE;
  hipStream_t stream = (hipStream_t)stream_;
  int device = 0;
  VL_HIP(hipGetDevice(&device));
  if (device < 0 || device >= 16) return VL_E_ARG;
  Scratch &s = g_scratch[device];
  std::lock_guard<std::mutex> lock(s.mu);
  WalkSpace *space = nullptr;
  Launch L;
  int32_t rc = space_of(s, stream, space);
  if (rc == VL_OK) rc = prepare_jobs(jobs, n_jobs, stream, *space, L, false, true);
  if (rc != VL_OK) return rc;
  if (L.maxK > kFewSamples) k_summarize<true><<<n_jobs, 1024, 0, stream>>>(L.dev, n_jobs, L.one, summaries, stats, L.finished);
  else k_summarize<false><<<(n_jobs + 3) / 4, 256, 0, stream>>>(L.dev, n_jobs, L.one, summaries, stats, L.finished);
  VL_HIP(hipGetLastError());
  return VL_OK;
}

namespace {
// the walk and the pair search over the job table L.dev with the board L.board
int32_t launch_all(const Launch &L, uint32_t n_jobs, hipStream_t stream, bool transposed, bool with_pairs) {
  const bool narrow = L.max_rows <= kPitchNarrow;   // every group of every job fits the narrow ring
  const size_t lds = (size_t)L.max_words * 64 * 4 + 64 * 4 + 1024 + (size_t)kRing * (narrow ? kPitchNarrow : kPitchWide) * 2;
  if (with_pairs && g_time_start) VL_HIP(hipEventRecord(g_time_start, stream));   // (the hook is for the verification calls)
  auto walk = [&](auto by_table, auto by_argument) {
    (n_jobs == 1 ? by_argument : by_table)<<<L.units, kWalkThreads, lds, stream>>>(L.one, L.dev, n_jobs, L.board);
  };
#define VL_WALK(...) walk(k_walk<__VA_ARGS__, false>, k_walk<__VA_ARGS__, true>)
  if (transposed) {
    if (narrow) VL_WALK(kPitchNarrow, true, false);
    else VL_WALK(kPitchWide, true, false);
  } else if (L.all_direct) {
    if (narrow) VL_WALK(kPitchNarrow, false, true);
    else VL_WALK(kPitchWide, false, true);
  } else {
    if (narrow) VL_WALK(kPitchNarrow, false, false);
    else VL_WALK(kPitchWide, false, false);
  }
#undef VL_WALK
  if (!with_pairs) {
    VL_HIP(hipGetLastError());
    return VL_OK;
  }
  if (g_time_stop) VL_HIP(hipEventRecord(g_time_stop, stream));
  g_time_start = g_time_stop = nullptr;
  VL_HIP(hipGetLastError());
  const uint32_t per_group = (uint32_t)std::min<uint64_t>(L.max_rows, std::max<uint64_t>(1, kResolveGroups / L.groups));
  (n_jobs == 1 ? L.shared ? k_resolve<true, true> : k_resolve<true, false> : L.shared ? k_resolve<false, true> : k_resolve<false, false>)
      <<<(uint32_t)L.groups * per_group, kResolveThreads, (size_t)L.max_w * 4, stream>>>(L.dev, n_jobs, L.one, per_group, (uint32_t)L.groups, L.board);
  VL_HIP(hipGetLastError());
  return VL_OK;
}

int32_t verify_jobs(const vl_job *jobs, uint32_t n_jobs, hipStream_t stream, bool transposed) {
  if (!jobs) return VL_E_NULL;
  if (n_jobs == 0 || n_jobs > 65535) return VL_E_SHAPE;
  int device = 0;
  VL_HIP(hipGetDevice(&device));
  if (device < 0 || device >= 16) return VL_E_ARG;
  Scratch &s = g_scratch[device];
  std::lock_guard<std::mutex> lock(s.mu);
  WalkSpace *space = nullptr;
  Launch L;
  int32_t rc = space_of(s, stream, space);
  if (rc == VL_OK) rc = prepare_jobs(jobs, n_jobs, stream, *space, L, transposed);
  if (rc != VL_OK) return rc;
  return launch_all(L, n_jobs, stream, transposed, true);
}
}  // namespace

int32_t vl::verdicts_only(const vl_job *jobs, uint32_t n_jobs, hipStream_t stream, WalkSpace &space) {
  Launch L;
  const int32_t rc = prepare_jobs(jobs, n_jobs, stream, space, L);
  if (rc != VL_OK) return rc;
  return launch_all(L, n_jobs, stream, false, false);
}

extern "C" int32_t vl_verify_multi(const vl_job *jobs, uint32_t n_jobs, vl_stream stream) {
  return verify_jobs(jobs, n_jobs, (hipStream_t)stream, false);
}

extern "C" int32_t vl_verify_multi_occ_major(const vl_job *jobs, uint32_t n_jobs, vl_stream stream) {
  return verify_jobs(jobs, n_jobs, (hipStream_t)stream, true);
}

extern "C" int32_t vl_verify_batch(const vl_mir *mir, const vl_live *live, const uint16_t *cand, uint32_t K,
                                   uint64_t ld, vl_result *out, vl_stream stream) {
  vl_job j = {mir, live, cand, K, ld, out};
  return vl_verify_multi(&j, 1, stream);
}

// ---- the entry point that allocates nothing ----------------------------------------------
// Its board lives in a file-scope device array instead of memory the library allocates.  The array's name is only a host-side handle:
// its device address is looked up once per device and kept.
namespace {
constexpr uint32_t kStaticMaxK = VL_STATIC_MAX_K;
struct StaticScratch {   // zero at load time, and between calls
  uint32_t head[kHeadWords];
  uint32_t arrived[kStaticMaxK];   // (a group may be a single row)
  uint32_t keys[kStaticMaxK];
};
}  // namespace
static __device__ __align__(256) unsigned char scratch[sizeof(StaticScratch)];
namespace {
std::mutex g_static_mu;
void *g_static_ptr[16] = {};
}  // namespace

extern "C" int32_t vl_verify_batch_static(const vl_mir *mir, const vl_live *live, const uint16_t *cand, uint32_t K,
                                          uint64_t ld, vl_result *out, vl_stream stream_) {
  if (K > kStaticMaxK) return VL_E_LIMIT;
  const vl_job u = {mir, live, cand, K, ld, out};
  DevJob d;
  Launch L;
  const int32_t rc = fill_jobs(&u, 1, false, &d, L);
  if (rc != VL_OK) return rc;
  hipStream_t stream = (hipStream_t)stream_;
  int device = 0;
  VL_HIP(hipGetDevice(&device));
  if (device < 0 || device >= 16) return VL_E_ARG;
  StaticScratch *sc;
  {
    // the array's address on this device, looked up on the first call made with it current
    std::lock_guard<std::mutex> lock(g_static_mu);
    if (!g_static_ptr[device]) {
      void *ptr = nullptr;
      VL_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
      g_static_ptr[device] = ptr;
    }
    sc = (StaticScratch *)g_static_ptr[device];
  }
  L.one = d;
  L.board = Board{sc->arrived, sc->keys};
  L.shared = true;
  return launch_all(L, 1, stream, false, true);
}
