"""Verification of many samples of a small program: a workgroup takes two or four of the analysis' short tiles
at once.  Joined or not, over tiles that end inside a block or at its start, with a last tile that has
no partner, in every layout: the oracle's results, exactly."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_2506_17506_amd as vl  # noqa: E402
from oracle import vlo  # noqa: E402
from vlgen import gen  # noqa: E402
from vlgen.mir import Mir  # noqa: E402
from test_gpu_parity import assert_results_equal, free  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    vl.load()


def results(out):
    return out.cpu().numpy().view(np.uint32).reshape(-1, 4).copy().view(vl.RESULT_DTYPE).reshape(-1)


def chain(n, seed):
    """blocks of 32 and 33 instructions: tiles of 32 start at block boundaries and inside"""
    rng = np.random.default_rng(seed)
    V = n // 2
    ins = [([v], [int(rng.integers(v))] if v else []) for v in range(V)] + [([], rng.integers(0, V, 2).tolist()) for _ in range(n - V)]
    ins = [(d, sorted(set(u))) for d, u in ins]
    cuts = [0]
    while cuts[-1] < n:
        cuts.append(min(n, cuts[-1] + (32 if len(cuts) % 3 else 33)))
    blocks = [ins[a:b] for a, b in zip(cuts, cuts[1:])]
    succ = [[b + 1] if b + 1 < len(blocks) else [] for b in range(len(blocks))]
    return Mir.build(blocks, succ, V, (512,), name=f"chain{n}")


def programs():
    for seed, (kind, n, damage) in enumerate([(gen.STRAIGHT, 200, 1), (gen.LOOP3, 610, 2)]):
        k = gen.Kernel(kind, 0x7A0 + seed, n, n if kind == gen.STRAIGHT else n * 3 // 4)
        yield k.mir, k.candidates(5, 90, 45, damage)[0]
    for n in (97, 330):
        m = chain(n, n)
        rng = np.random.default_rng(n)
        rows = np.zeros((90, m.n_occ), np.uint16)
        base = rng.integers(0, 512, (90, m.n_vreg))
        base[:60] = rng.permutation(512)[:m.n_vreg]
        rows[:] = base[:, m.occ_vreg]
        for r in range(20):
            rows[r, rng.integers(m.n_occ)] ^= 1
        yield m, rows


@pytest.mark.parametrize("K", [63, 8000, 20000])
def test_joined_tiles(K):
    tiles = 0
    for m, distinct in programs():
        an = vlo.analyze(m, threads=8)
        assert an.contract == 0
        which = np.random.default_rng(K).integers(0, len(distinct), K)
        want = vlo.verify(m, an, distinct, threads=8)[which]
        rows = np.ascontiguousarray(distinct[which])
        hm = vl.vl_mir_create(m)
        hl = vl.vl_liveness(hm)
        tiles = max(tiles, vl.vl_live_get(hl).n_tile * ((K + 63) // 64))
        try:
            dev, ld = vl.rows_to_device(rows)
            packed = torch.from_numpy(rows.view(np.int16)).cuda()
            pitch = (K + 7) // 8 * 8
            occ = torch.zeros((m.n_occ, pitch), dtype=torch.int16, device="cuda")
            occ[:, :K] = packed.t()
            for name, call in (
                    ("rows", lambda o: vl.vl_verify_batch(hm, hl, dev, K, ld, o)),
                    ("static", lambda o: vl.vl_verify_batch_static(hm, hl, dev, K, ld, o)),
                    ("packed", lambda o: vl.vl_verify_batch(hm, hl, packed, K, m.n_occ, o)),
                    ("occurrence-major", lambda o: vl.vl_verify_multi_occ_major([(hm, hl, occ, K, pitch, o)])),
                    ("two jobs", lambda o: vl.vl_verify_multi([(hm, hl, dev, K - 20, ld, o), (hm, hl, dev[K - 20:], 20, ld, o[K - 20:])]))):
                out = torch.full((K, 4), -1, dtype=torch.int32, device="cuda")
                call(out)
                torch.cuda.synchronize()
                assert_results_equal(want, results(out), f"{m.name} {name}")
        finally:
            free([hm], [hl])
    assert K < 100 or tiles > 1800   # (some of these join four)
