"""The analysis where its parts change shape: up to 32 blocks the fixed point keeps its rows in
registers, beyond that in LDS; counts are prefixed by stretches of 256 entries and instructions; the
tiles' live-ins are counted in windows of 2,048 tiles, by one workgroup for up to 1,024 words of vregs.
Everything against the oracle, exactly."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_2506_17506_amd as vl  # noqa: E402
from oracle import vlo  # noqa: E402
from vlgen.mir import Mir  # noqa: E402
from test_gpu_parity import assert_liveness_equal, assert_results_equal, free, gpu_analyze, gpu_verify  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    vl.load()


def flow_program(seed, n_block, n_vreg, per_block):
    """n_vreg values written in the entry block, then random reads and writes in blocks joined by random
    edges, forwards and backwards, none to four more out of each"""
    rng = np.random.default_rng(seed)
    entry = [(list(range(v, min(n_vreg, v + 30))), []) for v in range(0, n_vreg, 30)]
    blocks = [entry + [([], [int(rng.integers(n_vreg))])]]
    for _ in range(n_block - 1):
        blocks.append([(rng.integers(0, n_vreg, rng.integers(0, 3)).tolist(), np.unique(rng.integers(0, n_vreg, 1 + rng.integers(0, 3))).tolist())
                       for _ in range(1 + int(rng.integers(per_block)))])
    for blk in blocks:
        for x, (d, u) in enumerate(blk):
            blk[x] = (sorted(set(d)), u)
    succ = []
    for b in range(n_block):
        more = rng.integers(0, n_block, rng.integers(0, 5)) if rng.random() < 0.6 else np.zeros(0, int)
        succ.append(sorted({*([b + 1] if b + 1 < n_block else []), *[int(x) for x in more]}))
    return Mir.build(blocks, succ, n_vreg, (512,), name=f"flow{n_block}x{n_vreg}")


def check(mirs, tile_len=0, dense=True):
    hm, hl, got, _ = gpu_analyze(mirs, tile_len, dense)
    try:
        rows_list, wants = [], []
        rng = np.random.default_rng(3)
        for m, g in zip(mirs, got):
            an = vlo.analyze(m, threads=8)
            assert an.contract == 0
            assert_liveness_equal(m, an, g, m.name)
            rows = rng.integers(0, 512, (3, m.n_vreg)).astype(np.uint16)[:, m.occ_vreg]
            rows_list.append(np.ascontiguousarray(rows))
            wants.append(vlo.verify(m, an, rows_list[-1], threads=8))
        for m, w, r in zip(mirs, wants, gpu_verify(hm, hl, rows_list)):
            assert_results_equal(w, r, m.name)
    finally:
        free(hm, hl)


@pytest.mark.parametrize("n_block", [1, 2, 3, 31, 32, 33, 40])
@pytest.mark.parametrize("n_vreg", [1, 33, 2048, 2100])
def test_blocks_around_the_registers(n_block, n_vreg):
    check([flow_program(n_block * 10000 + n_vreg, n_block, n_vreg, 8)])


def test_batch_on_both_sides():
    """a batch takes the way of its largest program; small ones beside it end early"""
    check([flow_program(s, b, v, 6) for s, b, v in ((1, 32, 700), (2, 1, 5), (3, 7, 64), (4, 20, 3000))])
    check([flow_program(s, b, v, 6) for s, b, v in ((1, 45, 300), (2, 1, 5), (3, 32, 64))])


@pytest.mark.parametrize("n", [255, 256, 257, 511, 513])
def test_stretches(n):
    """n instructions of one operand each, then of two"""
    for width in (1, 2):
        blk = [([0, 1][:width], [])] + [([], [0, 1][:width]) for _ in range(n - 1)]
        cut = n // 2
        check([Mir.build([blk[:cut], blk[cut:]], [[1], []], 2, (512,), name=f"n{n}x{width}")])


@pytest.mark.parametrize("tile_len", [1, 3])
def test_many_tiles(tile_len):
    """more tiles than a window counts (2,048)"""
    check([flow_program(77, 12, 90, 900)], tile_len, dense=False)


@pytest.mark.parametrize("n_vreg", [32 * 1024, 32 * 1024 + 1, 70000])
def test_wide_rows(n_vreg):
    """around the 1,024 words that one workgroup takes"""
    check([flow_program(5, 4, n_vreg, 40), flow_program(6, 9, 50, 30)], dense=False)


def with_gaps(m, step):
    """the program with its vregs numbered `step` apart: those in between are never mentioned"""
    V = m.n_vreg * step
    return Mir(m.blk_start, m.succ_off, m.succ, m.instr_occ_off, m.occ_vreg * np.uint32(step), m.occ_flags,
               np.zeros(V, np.uint8), np.ones(V, np.uint8), np.ones(V, np.uint8), m.class_size, None, name=f"{m.name}_by{step}")


@pytest.mark.parametrize("n_block,step", [(1, 4), (2, 16), (3, 64)])
def test_gaps_in_the_numbering_beside_a_program_of_many_blocks(n_block, step):
    """1,024 entries of the small program span more bitset words than they could without gaps, and the
    other program's blocks make room for a table of that many: the block sets are collected there, in new
    handles and in recycled ones (whose sizes are not read back)"""
    rng = np.random.default_rng(step)
    V = 700
    defs = [([v], []) for v in range(V)]
    reads = [([], sorted(set(rng.integers(0, V, 2).tolist()))) for _ in range(V)]
    cut = np.linspace(0, len(reads), n_block + 1).astype(int)
    blocks = [(defs if b == 0 else []) + reads[cut[b]:cut[b + 1]] for b in range(n_block)]
    succ = [[b + 1] if b + 1 < n_block else [] for b in range(n_block)]
    small = with_gaps(Mir.build(blocks, succ, V, (512,), name=f"gaps{n_block}"), step)
    mirs = [flow_program(1, 22, 34 * 32, 8), small, flow_program(2, 22, 40 * 32, 8)]
    ans = [vlo.analyze(m, threads=8) for m in mirs]
    assert all(an.contract == 0 for an in ans)
    hm, hl, got, _ = gpu_analyze(mirs)
    try:
        for _ in range(2):
            for m, an, g in zip(mirs, ans, got):
                assert_liveness_equal(m, an, g, m.name)
            hl = vl.vl_liveness_multi(hm, vl.VL_DENSE_POINTS, live=hl)
            torch.cuda.synchronize()
            got = [vl.view_to_numpy(vl.vl_live_get(h)) for h in hl]
        for m, an, g in zip(mirs, ans, got):
            assert_liveness_equal(m, an, g, m.name)
    finally:
        free(hm, hl)


def test_programs_around_what_the_host_derives():
    """arrays that follow from the description are written by the host for up to 11,500 instructions, vregs and
    occurrences together, by the device beyond: the same program a little smaller and a little larger"""
    from vlgen.mixed import mixed_mir
    sides = set()
    for seed, n in ((1, 200), (2, 1500), (3, 1900), (4, 2100), (5, 2300), (6, 2600), (7, 4000)):
        m = mixed_mir(0xB700 + seed, n_instr=n, reserved=seed % 2 == 0)
        V, O = m.n_vreg, m.n_occ
        rng = np.random.default_rng(seed)
        # early-clobber definitions here and there
        m.occ_flags[(m.occ_flags & 1 == 1) & (rng.random(O) < 0.1)] |= 4
        sides.add((n + V + O <= 11500))
        check([m])
    assert sides == {True, False}
    last = [flow_program(8, 5, v, 300) for v in (500, 3000, 6000)]
    check(last)


@pytest.mark.parametrize("n, n_block", [(8, 5), (9, 5), (16, 5), (48, 3), (48, 40), (163, 2)])
@pytest.mark.parametrize("alike", [True, False])
def test_batches_dealt_out_to_the_dies(n, n_block, alike):
    """programs alike (eight and multiples: dealt out evenly; 163: rows of eight, the last of three) and of mixed
    sizes (dealt out where to and fro leaves the dies equally busy)"""
    rng = np.random.default_rng(n)
    check([flow_program(k, n_block, 40 if alike else int(rng.integers(20, 400)), 8 if alike else 3 + k % 7) for k in range(n)], dense=n % 16 == 0)


def test_many_entries_beside_the_sort_for_large_programs():
    """a batch of more than half a million occurrences (entries put in order by workgroups of 512 threads) with programs of more
    vregs than are counted in LDS, whose lists are sorted in launches of their own"""
    large, small = flow_program(21, 4, 33000, 900), flow_program(22, 5, 60, 40)
    mirs = [large, small] + [large] * 15
    assert sum(-(-m.n_occ // 256) for m in mirs) // 4 > 512 and large.n_vreg > 32768
    ans = {id(m): vlo.analyze(m, interference=False, threads=8) for m in (large, small)}
    hm, hl, got, _ = gpu_analyze(mirs, dense=False)
    try:
        for m, g in zip(mirs, got):
            assert_liveness_equal(m, ans[id(m)], g, m.name)
    finally:
        free(hm, hl)
