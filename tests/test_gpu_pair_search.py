"""The pair search of the verifier with many values live at once and with every
row of a group failing, against the oracle, exactly."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_2506_17506_amd as vl  # noqa: E402
from oracle import vlo  # noqa: E402
from vlgen.mir import Mir  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    vl.load()


@pytest.mark.parametrize("n_live", [1, 64, 511, 512, 513, 800])
@pytest.mark.parametrize("K", [1, 64, 129])
def test_many_live_values(n_live, K):
    check_many_live_values(n_live, K, 0)


@pytest.mark.parametrize("n_live", [127, 128, 129, 383, 384, 385, 510, 511, 512, 800])
@pytest.mark.parametrize("tile_len", [100, 4096])
def test_lists_longer_than_a_thread_keeps(n_live, tile_len):
    """live-in lists around the 128 entries and tiles around the 384 events that the search keeps in registers,
    and around the 512 values that it lists of longer ones"""
    check_many_live_values(n_live, 64, tile_len)


def check_many_live_values(n_live, K, tile_len):
    """n_live values of two files live together; the last one written clashes in almost every row"""
    rng = np.random.default_rng(n_live)
    V = n_live + 1
    vclass = (np.arange(V) % 2).astype(np.uint8)
    blocks = [[([v], []) for v in range(V)] + [([], list(range(v, min(V, v + 40)))) for v in range(0, V, 40)]]
    m = Mir.build(blocks, [[]], V, (512, 512), vclass, np.ones(V, np.uint8), np.ones(V, np.uint8), None, name=f"live{n_live}")
    table = np.zeros((K, V), np.int64)
    for k in range(K):
        for c in (0, 1):
            mine = np.nonzero(vclass == c)[0]
            table[k, mine] = rng.permutation(512)[:len(mine)]
        if n_live and k % 8:
            same = np.nonzero(vclass[:n_live] == vclass[n_live])[0]
            if len(same):
                table[k, n_live] = table[k, rng.choice(same)]
    rows = np.ascontiguousarray(table[:, m.occ_vreg].astype(np.uint16))
    an = vlo.analyze(m)
    want = vlo.verify(m, an, rows)
    if 64 <= n_live <= 800 and K > 1:
        assert (want["status"] == 3).sum() > K // 2
    hm = vl.vl_mir_create(m)
    hl = vl.vl_liveness_multi([hm], tile_len=tile_len)[0]
    try:
        dev, ld = vl.rows_to_device(rows)
        out = torch.full((K, 4), -1, dtype=torch.int32, device="cuda")
        for _ in range(2):   # the second call finds the library's workspace as the first left it
            out.fill_(-1)
            vl.vl_verify_batch(hm, hl, dev, K, ld, out)
            torch.cuda.synchronize()
            got = out.cpu().numpy().view(np.uint32).copy().view(vl.RESULT_DTYPE).reshape(-1)
            bad = np.nonzero(want != got)[0]
            assert len(bad) == 0, f"row {bad[0]}: oracle {want[bad[0]]} gpu {got[bad[0]]}"
    finally:
        vl.vl_live_destroy(hl)
        vl.vl_mir_destroy(hm)
