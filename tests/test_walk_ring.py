"""What the lanes of the verifier's check wavefronts read of the LDS ring while the next chunk is being
written into it (vl_dev.h), compiled for the host.

While chunk c is checked, the same wavefronts write chunk c + 1 over the oldest of the ring's three
chunks, with no barrier in between: no lane may read a slot of chunk c + 1 then, those with nothing to
check included."""
import subprocess

import pytest

from stand_in import ROOT

SOURCE = """
#include <cstdio>
#include "vl_dev.h"
using namespace vl;
int main() {
  // a lane outside the tile: [0, lead) in a tile's first chunk, for every place a tile can start, and the lanes behind its last
  unsigned tiles = 0, overlaps = 0, verdicts = 0;
  for (uint32_t oa = 0; oa < 4096; ++oa) {
    if (oa % kWalkChunk == 0) continue;
    const uint32_t c = oa / kWalkChunk;
    ++tiles;
    bool meets = false;
    for (uint32_t lane = 0; lane < kWalkChunk; ++lane) {
      const u32x4 r = nothing_to_check(c, lane);
      // as the walk takes the record apart: it reads one slot twice (no kChkNear), and must find nothing wrong in any value
      const uint32_t slot = (r.x >> 8) & 0xFFFu, next = (c + 1) % (kWalkRing / kWalkChunk) * kWalkChunk;
      meets |= slot >= next && slot < next + kWalkChunk;
      if ((r.x & 0xFFu) != 0 || r.y != 0 || r.z != 0 || r.w != 0xFFFFFFFFu) ++verdicts;
    }
    overlaps += meets;
  }
  // a link counts as near from here on: the slot of an earlier occurrence is read for it
  for (uint32_t o = 0; o < 4096; ++o)
    for (uint32_t prev = o < 400 ? 0 : o - 400; prev < o; ++prev)
      if (check_reaches(o, prev)) {
        const uint32_t slot = prev % kWalkRing, next = (o / kWalkChunk + 1) % (kWalkRing / kWalkChunk) * kWalkChunk;
        if (slot >= next && slot < next + kWalkChunk) ++overlaps;
      }
  printf("tiles %u overlaps %u verdicts %u\\n", tiles, overlaps, verdicts);
  return overlaps || verdicts;
}
"""


def test_nothing_that_is_being_written_is_read(tmp_path):
    src, exe = tmp_path / "ring.hip", tmp_path / "ring"
    src.write_text(SOURCE)
    subprocess.run(["hipcc", "--cuda-host-only", "-O1", "-std=c++17", "-I", f"{ROOT}/paper_2506_17506_amd/csrc", "-o", str(exe), str(src)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
    assert "tiles 4032" in r.stdout
