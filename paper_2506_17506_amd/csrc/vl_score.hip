// Register-bank conflicts of candidates, a quality measure beside validity (Section 2:
// registers are organised in banks, four on NVIDIA GPUs; reading several values from one
// bank stalls the pipeline a cycle per extra value).  A workgroup takes 256 instructions, one per
// lane, and a slab of candidates.  What does not depend on the candidate is found once: for every
// operand, the width of its vreg if the operand is the first USE of that vreg in its
// instruction, else 0.  The lanes of a wavefront, being neighbouring instructions, read
// neighbouring entries of a candidate row.  For every bank the registers read from it are
// counted in closed form from base and width; the worst bank gives the stall.
#include "vl_dev.h"

using namespace vl;

namespace {

// how many of the registers p .. p + w - 1 lie in bank b of n: w / n, and one more in the w % n banks
// from p % n on
__device__ inline uint32_t in_bank(uint32_t p_mod, uint32_t w_div, uint32_t w_mod, uint32_t b, uint32_t n) {
  return w_div + ((b >= p_mod ? b - p_mod : b + n - p_mod) < w_mod ? 1u : 0u);
}

constexpr uint32_t kScoreInstr = 256;   // instructions per workgroup, one per lane
constexpr uint32_t kScoreCands = 4;     // candidates per workgroup
constexpr uint32_t kScoreFew = 4;       // operands an instruction usually has at most

// the four banks' counts are four 16-bit fields of one word: a tuple of width w at base p adds
// w / 4 to every bank and one more to the w % 4 banks from p % 4 on (a rotation of the field
// pattern); at most 64 x 9 per bank
__device__ inline uint64_t four_banks(uint32_t w, uint32_t p) {
  const uint32_t rest = w & 3u, sh = (p & 3u) * 16u;
  const uint64_t ones = 0x0000000100010001ull & ((1ull << (16u * rest)) - 1ull);
  return (uint64_t)(w >> 2) * 0x0001000100010001ull + ((ones << sh) | (ones >> ((64u - sh) & 63u) & (sh ? ~0ull : 0ull)));
}
__device__ inline uint32_t worst_of(uint64_t counts) {
  const uint32_t lo = (uint32_t)counts, hi = (uint32_t)(counts >> 32);
  return max(max(lo & 0xFFFFu, lo >> 16), max(hi & 0xFFFFu, hi >> 16));
}

// One, two, four and eight banks with up to four operands: counts fit bytes (4 x 32 at most), one per bank, the
// pattern of one or two banks repeated over four.  The bytes stand for the banks in descending order (which bank is
// the worst does not matter), so that a tuple of width w at base p adds w / n everywhere and a pattern that depends on
// w % n, rotated to the right by p bytes.
struct Pattern { uint32_t lo, hi; };   // (eight banks: bytes 4..7 in hi)
__device__ inline Pattern pattern_of(uint32_t w, uint32_t n) {   // bytes 0, -1, -2, ... (modulo n) of w % n banks
  const uint32_t rest = w & (n - 1u);
  if (n == 8) {
    const uint64_t x = rest ? 1ull | (rest > 1u ? 0x0101010101010101ull << (8u * (9u - rest)) : 0ull) : 0ull;
    return {(uint32_t)x, (uint32_t)(x >> 32)};
  }
  if (n == 4) return {rest ? 1u | (rest > 1u ? 0x01010101u << (8u * (5u - rest)) : 0u) : 0u, 0u};
  return {rest ? 0x00010001u : 0u, 0u};
}
__device__ inline uint32_t worst_byte(uint32_t a, uint32_t b) {   // of eight
  typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
  auto pairs = [](uint32_t x) { return __builtin_elementwise_max(__builtin_bit_cast(u16x2, x & 0x00FF00FFu), __builtin_bit_cast(u16x2, (x >> 8) & 0x00FF00FFu)); };
  const u16x2 m = __builtin_elementwise_max(pairs(a), pairs(b));
  return max((uint32_t)m.x, (uint32_t)m.y);
}

// sum over the wavefront, in its last lane (rows of 16 lanes, then across rows)
__device__ inline uint32_t wave_total(uint32_t x) {
  x += __builtin_amdgcn_update_dpp(0u, x, 0x111, 0xf, 0xf, false);   // row_shr:1, 2, 4, 8
  x += __builtin_amdgcn_update_dpp(0u, x, 0x112, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0u, x, 0x114, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0u, x, 0x118, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0u, x, 0x142, 0xa, 0xf, false);   // row_bcast:15 into rows 1 and 3
  x += __builtin_amdgcn_update_dpp(0u, x, 0x143, 0xc, 0xf, false);   // row_bcast:31 into rows 2 and 3
  return x;
}

// What bounds it: waiting for memory.  A lane's operands are a chain of reads (offsets, records,
// attributes), and a register per operand and candidate, which needs the offsets alone: for an instruction with at
// most four operands the 4 x 4 reads of a slab go out together with the records (a loop
// over the operands waited for each: 35 us for 10,000 instructions and 100 candidates; registers read behind the
// attributes, counts in 16-bit fields of 64 bits and sums by shuffles through LDS, which a single longer
// instruction made the whole launch wait for: 13.2; 9.4 this way, 9.7 with slabs of eight, 10.3 of five).
// kBytes: one, two, four or eight banks.
template <bool kBytes>
__global__ __launch_bounds__(256) void k_bank_score(const DevMir *mir, const uint16_t *__restrict__ cand, uint32_t K, uint64_t ld,
                                                    uint32_t n_banks, uint32_t *__restrict__ out) {
  const DevMir VL_GLOBAL &m = *as_global(mir);
  __shared__ uint32_t sums[kScoreCands];
  const uint32_t i = blockIdx.x * kScoreInstr + threadIdx.x;
  const uint32_t k0 = blockIdx.y * kScoreCands, kn = min(kScoreCands, K - k0);
  if (threadIdx.x < kScoreCands) sums[threadIdx.x] = 0;
  const uint32_t o0 = i < m.N ? m.occ_off[i] : 0u, o1 = i < m.N ? m.occ_off[i + 1] : 0u, n = o1 - o0;
  const uint16_t VL_GLOBAL *rows = as_global(cand) + (uint64_t)k0 * ld;
  uint32_t stall[kScoreCands];
#pragma unroll
  for (uint32_t c = 0; c < kScoreCands; ++c) stall[c] = 0;
  __syncthreads();
  {
    const uint32_t few = n <= kScoreFew ? n : 0u;   // (longer instructions follow)
    uint64_t rec[kScoreFew];
    uint32_t p[kScoreCands][kScoreFew], v[kScoreFew], w[kScoreFew];
#pragma unroll
    for (uint32_t u = 0; u < kScoreFew; ++u) rec[u] = u < few ? m.occ_rec[o0 + u] : 0ull;
#pragma unroll
    for (uint32_t c = 0; c < kScoreCands; ++c)
#pragma unroll
      for (uint32_t u = 0; u < kScoreFew; ++u) p[c][u] = c < kn && u < few ? rows[c * ld + o0 + u] : 0u;
#pragma unroll
    for (uint32_t u = 0; u < kScoreFew; ++u) v[u] = (rec[u] >> 32) & VL_OCC_USE ? (uint32_t)rec[u] & ~kRecKeeps : kNone;
#pragma unroll
    for (uint32_t u = 0; u < kScoreFew; ++u) {
      bool read = v[u] != kNone;
#pragma unroll
      for (uint32_t x = 0; x < u; ++x) read &= v[x] != v[u];   // the first USE of the vreg in its instruction
      w[u] = read ? attr_width(m.vattr[v[u]]) : 0u;
    }
    if constexpr (kBytes) {
      Pattern pat[kScoreFew];
      uint32_t all = 0;
#pragma unroll
      for (uint32_t u = 0; u < kScoreFew; ++u) {
        all += (w[u] >> __builtin_ctz(n_banks)) * 0x01010101u;
        pat[u] = pattern_of(w[u], n_banks);
      }
      const bool eight = n_banks == 8;
#pragma unroll
      for (uint32_t c = 0; c < kScoreCands; ++c) {
        uint32_t lo = all, hi = all;
#pragma unroll
        for (uint32_t u = 0; u < kScoreFew; ++u) {
          const uint32_t s = p[c][u] * 8u;   // (the rotation takes it modulo 32)
          if (!eight) {
            lo += __builtin_amdgcn_alignbit(pat[u].lo, pat[u].lo, s);
          } else {
            const bool swap = (p[c][u] & 4u) != 0;
            const uint32_t a = swap ? pat[u].hi : pat[u].lo, b = swap ? pat[u].lo : pat[u].hi;
            lo += __builtin_amdgcn_alignbit(b, a, s);
            hi += __builtin_amdgcn_alignbit(a, b, s);
          }
        }
        const uint32_t worst = worst_byte(lo, eight ? hi : lo);
        stall[c] = worst > 1 ? worst - 1 : 0;
      }
    } else {
      uint32_t w_div[kScoreFew], w_mod[kScoreFew];
#pragma unroll
      for (uint32_t u = 0; u < kScoreFew; ++u) { w_div[u] = w[u] / n_banks; w_mod[u] = w[u] % n_banks; }
#pragma unroll
      for (uint32_t c = 0; c < kScoreCands; ++c) {
        uint32_t worst = 0, p_mod[kScoreFew];
#pragma unroll
        for (uint32_t u = 0; u < kScoreFew; ++u) p_mod[u] = p[c][u] % n_banks;
        for (uint32_t b = 0; b < n_banks; ++b) {
          uint32_t reads = 0;
#pragma unroll
          for (uint32_t u = 0; u < kScoreFew; ++u) reads += in_bank(p_mod[u], w_div[u], w_mod[u], b, n_banks);
          worst = max(worst, reads);
        }
        stall[c] = worst > 1 ? worst - 1 : 0;
      }
    }
  }
  // longer instructions, one after the other: an operand per lane (at most 64)
  for (uint64_t todo = __ballot(n > kScoreFew); todo; todo &= todo - 1) {
    const uint32_t at = (uint32_t)__builtin_ctzll(todo), lane = threadIdx.x & 63u;
    const uint32_t first = __builtin_amdgcn_readlane(o0, at), n_ops = __builtin_amdgcn_readlane(n, at);
    const uint64_t rec = lane < n_ops ? m.occ_rec[first + lane] : 0ull;
    uint32_t p[kScoreCands];
#pragma unroll
    for (uint32_t c = 0; c < kScoreCands; ++c) p[c] = c < kn && lane < n_ops ? rows[c * ld + first + lane] : 0u;
    const uint32_t v = (rec >> 32) & VL_OCC_USE ? (uint32_t)rec & ~kRecKeeps : kNone;
    bool read = v != kNone;
    for (uint32_t x = 0; x < n_ops; ++x) {
      const uint32_t other = __builtin_amdgcn_readlane(v, x);
      read &= (x >= lane) | (other != v);
    }
    const uint32_t w = read ? attr_width(m.vattr[v]) : 0u;
    auto total = [](uint32_t x) { return (uint32_t)__builtin_amdgcn_readlane(wave_total(x), 63); };
#pragma unroll
    for (uint32_t c = 0; c < kScoreCands; ++c) {
      uint32_t worst = 0;
      if (kBytes && n_banks == 4) {
        const uint64_t counts = four_banks(w, p[c]);
        worst = worst_of((uint64_t)total((uint32_t)counts) | ((uint64_t)total((uint32_t)(counts >> 32)) << 32));
      } else {
        for (uint32_t b = 0; b < n_banks; ++b) worst = max(worst, total(in_bank(p[c] % n_banks, w / n_banks, w % n_banks, b, n_banks)));
      }
      if (lane == at) stall[c] = worst > 1 ? worst - 1 : 0;
    }
  }
#pragma unroll
  for (uint32_t c = 0; c < kScoreCands; ++c) {
    const uint32_t total = wave_total(stall[c]);
    if ((threadIdx.x & 63u) == 63u && total) atomicAdd(&sums[c], total);
  }
  __syncthreads();
  if (threadIdx.x < kn && sums[threadIdx.x]) atomicAdd(&out[k0 + threadIdx.x], sums[threadIdx.x]);
}

__global__ void k_score_clear(uint32_t *out, uint32_t K) {
  const uint32_t k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k < K) out[k] = 0;
}

}  // namespace

extern "C" int32_t vl_bank_conflicts(const vl_mir *mir, const uint16_t *cand, uint32_t K, uint64_t ld, uint32_t n_banks,
                                     uint32_t *out, vl_stream stream_) {
  if (!mir || !cand || !out) return VL_E_NULL;
  if (mir->magic != kMirMagic || mir->lowered) return VL_E_ARG;
  if (K == 0 || K > 65535 || ld < mir->h.O) return VL_E_SHAPE;
  if (n_banks == 0 || n_banks > 64) return VL_E_RANGE;
  hipStream_t stream = (hipStream_t)stream_;
  k_score_clear<<<(K + 255) / 256, 256, 0, stream>>>(out, K);
  const dim3 grid((mir->h.N + kScoreInstr - 1) / kScoreInstr, (K + kScoreCands - 1) / kScoreCands);
  (n_banks <= 8 && (n_banks & (n_banks - 1)) == 0 ? k_bank_score<true> : k_bank_score<false>)<<<grid, 256, 0, stream>>>(mir->dev, cand, K, ld, n_banks, out);
  VL_HIP(hipGetLastError());
  return VL_OK;
}
