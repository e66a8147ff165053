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
constexpr uint32_t kScoreCands = 8;     // candidates per workgroup
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

// What bounds it: waiting for memory.  A lane's operands are a chain of reads (offsets, vregs,
// attributes) done once, and then a register per operand and candidate; for an instruction with at
// most four operands the 8 x 4 reads of a slab are independent and all in flight together (a loop
// over the operands waited for each: 35 us for 10,000 instructions and 100 candidates).
template <bool kFour>
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
    uint32_t v[kScoreFew], w[kScoreFew];
#pragma unroll
    for (uint32_t u = 0; u < kScoreFew; ++u) v[u] = u < few && (m.occ_flags[o0 + u] & VL_OCC_USE) ? m.occ_vreg[o0 + u] : kNone;
#pragma unroll
    for (uint32_t u = 0; u < kScoreFew; ++u) {
      bool read = v[u] != kNone;
#pragma unroll
      for (uint32_t x = 0; x < u; ++x) read &= v[x] != v[u];   // the first USE of the vreg in its instruction
      w[u] = read ? attr_width(m.vattr[v[u]]) : 0u;
    }
    uint32_t w_div[kScoreFew], w_mod[kScoreFew];
    if (!kFour)
#pragma unroll
      for (uint32_t u = 0; u < kScoreFew; ++u) { w_div[u] = w[u] / n_banks; w_mod[u] = w[u] % n_banks; }
    uint32_t p[kScoreCands][kScoreFew];
#pragma unroll
    for (uint32_t c = 0; c < kScoreCands; ++c)
#pragma unroll
      for (uint32_t u = 0; u < kScoreFew; ++u) p[c][u] = c < kn && w[u] ? rows[c * ld + o0 + u] : 0u;
#pragma unroll
    for (uint32_t c = 0; c < kScoreCands; ++c) {
      uint32_t worst = 0;
      if (kFour) {
        uint64_t counts = 0;
#pragma unroll
        for (uint32_t u = 0; u < kScoreFew; ++u) counts += four_banks(w[u], p[c][u]);
        worst = worst_of(counts);
      } else {
        uint32_t p_mod[kScoreFew];
#pragma unroll
        for (uint32_t u = 0; u < kScoreFew; ++u) p_mod[u] = p[c][u] % n_banks;
        for (uint32_t b = 0; b < n_banks; ++b) {
          uint32_t reads = 0;
#pragma unroll
          for (uint32_t u = 0; u < kScoreFew; ++u) reads += in_bank(p_mod[u], w_div[u], w_mod[u], b, n_banks);
          worst = max(worst, reads);
        }
      }
      stall[c] = worst > 1 ? worst - 1 : 0;
    }
  }
  // longer instructions, one after the other: an operand per lane (at most 64)
  for (uint64_t todo = __ballot(n > kScoreFew); todo; todo &= todo - 1) {
    const uint32_t at = (uint32_t)__builtin_ctzll(todo), lane = threadIdx.x & 63u;
    const uint32_t first = __builtin_amdgcn_readlane(o0, at), n_ops = __builtin_amdgcn_readlane(n, at);
    const uint32_t v = lane < n_ops && (m.occ_flags[first + lane] & VL_OCC_USE) ? m.occ_vreg[first + lane] : kNone;
    bool read = v != kNone;
    for (uint32_t x = 0; x < n_ops; ++x) {
      const uint32_t other = __builtin_amdgcn_readlane(v, x);
      read &= (x >= lane) | (other != v);
    }
    const uint32_t w = read ? attr_width(m.vattr[v]) : 0u;
    uint32_t p[kScoreCands];
#pragma unroll
    for (uint32_t c = 0; c < kScoreCands; ++c) p[c] = c < kn && w ? rows[c * ld + first + lane] : 0u;
#pragma unroll
    for (uint32_t c = 0; c < kScoreCands; ++c) {
      uint32_t worst = 0;
      if (kFour) {
        uint64_t counts = four_banks(w, p[c]);
        for (int d = 32; d >= 1; d >>= 1) counts += __shfl_xor(counts, d, 64);
        worst = worst_of(counts);
      } else {
        for (uint32_t b = 0; b < n_banks; ++b) {
          uint32_t reads = in_bank(p[c] % n_banks, w / n_banks, w % n_banks, b, n_banks);
          for (int d = 32; d >= 1; d >>= 1) reads += (uint32_t)__shfl_xor((int)reads, d, 64);
          worst = max(worst, reads);
        }
      }
      if (lane == at) stall[c] = worst > 1 ? worst - 1 : 0;
    }
  }
#pragma unroll
  for (uint32_t c = 0; c < kScoreCands; ++c) {
    for (int d = 32; d >= 1; d >>= 1) stall[c] += (uint32_t)__shfl_xor((int)stall[c], d, 64);
    if ((threadIdx.x & 63u) == 0 && stall[c]) atomicAdd(&sums[c], stall[c]);
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
  (n_banks == 4 ? k_bank_score<true> : k_bank_score<false>)<<<grid, 256, 0, stream>>>(mir->dev, cand, K, ld, n_banks, out);
  VL_HIP(hipGetLastError());
  return VL_OK;
}
