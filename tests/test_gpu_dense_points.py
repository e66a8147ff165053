"""The dense per-point sets around the 64 instructions and 64 bitset words a workgroup takes at a
time, against the oracle, bit for bit."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_2506_17506_amd as vl  # noqa: E402
from oracle import vlo  # noqa: E402
from vlgen import gen  # noqa: E402
from vlgen.mixed import many_blocks_mir, mixed_mir  # noqa: E402
from test_gpu_parity import assert_liveness_equal, free, gpu_analyze  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    vl.load()


@pytest.mark.parametrize("tile_len", [0, 16, 63, 64, 65, 128, 200, 5000])   # (16: a launch of its own)
def test_tile_and_row_edges(tile_len):
    # 47 words; 64 and 65 words; mixed shapes; a chain of 60 blocks
    mirs = [gen.Kernel(gen.LOOP3, 0x2D0, 2000, 1500).mir, gen.Kernel(gen.STRAIGHT, 0x2D1, 64 * 32, 64 * 32).mir,
            gen.Kernel(gen.STRAIGHT, 0x2D2, 64 * 32 + 1, 64 * 32 + 1).mir, mixed_mir(0xD300, n_instr=700, early=0.3),
            many_blocks_mir(3, n_blocks=60, per=20)]
    ans = [vlo.analyze(m, interference=False, threads=8) for m in mirs]
    keep = [k for k, a in enumerate(ans) if a.contract == 0]
    assert len(keep) >= 4
    mirs, ans = [mirs[k] for k in keep], [ans[k] for k in keep]
    hm, hl, got, _ = gpu_analyze(mirs, tile_len)
    try:
        for m, an, g in zip(mirs, ans, got):
            assert_liveness_equal(m, an, g, f"{m.name} tile {tile_len}")
    finally:
        free(hm, hl)
