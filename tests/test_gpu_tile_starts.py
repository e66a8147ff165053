"""Tiles that start inside a chunk of 64 occurrences whose successor takes the ring's first slots: the lanes of the
occurrences before such a tile have nothing to check, while the chunk after theirs is being written
(test_walk_ring.py).  Every verdict against the oracle, and no broken rule without its name."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_2506_17506_amd as vl  # noqa: E402
from oracle import vlo  # noqa: E402
from vlgen import gen  # noqa: E402
from test_gpu_parity import assert_results_equal, free, gpu_analyze, gpu_verify  # noqa: E402
from test_gpu_occ_major import verify_occ_major  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    vl.load()


@pytest.mark.parametrize("damaged", [0.0, 0.5])
@pytest.mark.parametrize("K", [50, 64])   # either pitch of the ring
def test_tiles_that_start_before_the_rings_first_slots(K, damaged):
    kernels = [gen.Kernel((gen.MHA, gen.GEMM)[s % 2], 0x715 + s, 2500, 1900) for s in range(8)]
    rows = [k.candidates(77 + s, K, int(K * damaged), 2)[0] for s, k in enumerate(kernels)]
    mirs = [k.mir for k in kernels]
    want = [vlo.verify(m, vlo.analyze(m), r) for m, r in zip(mirs, rows)]
    for tile_len in (61, 128):
        start = [m.instr_occ_off[np.minimum(np.arange(0, m.n_instr + tile_len, tile_len), m.n_instr)].astype(int) for m in mirs]
        meant = sum(int(((s[:-1] % 64 != 0) & (s[:-1] // 64 % 3 == 2) & ((s[1:] - 1) // 64 > s[:-1] // 64)).sum()) for s in start)
        assert meant > 30, meant
        hm, hl, _, _ = gpu_analyze(mirs, tile_len, dense=False)
        try:
            for _ in range(5):
                for how in (True, False, "occurrence-major"):
                    got = verify_occ_major(hm, hl, rows) if how == "occurrence-major" else gpu_verify(hm, hl, rows, how)
                    for k in range(len(mirs)):
                        assert not ((got[k]["status"] == 2) & (got[k]["b"] == 0)).any()
                        assert_results_equal(want[k], got[k], f"kernel {k} tile {tile_len} rows {how}")
        finally:
            free(hm, hl)
