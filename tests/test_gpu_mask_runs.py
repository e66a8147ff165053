"""Decoding masks where neighbouring queries fold into runs: many rows of one occurrence at equal
and unequal distances, more runs than travel as a kernel argument (64), shares of several
queries per wavefront, more than 256 live values; against the oracle, bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_2506_17506_amd as vl  # noqa: E402
from oracle import vlo  # noqa: E402
from vlgen import gen  # noqa: E402
from vlgen.mir import Mir  # noqa: E402
from vlgen.mixed import mixed_mir  # noqa: E402
from test_gpu_parity import free, gpu_analyze  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    vl.load()


def orders(n_rows, occs, rng):
    """row order and occurrence of every query, as (name, [(row, occ)])"""
    yield "one run each", [(k, o) for o in occs[:3] for k in range(n_rows)]
    yield "backwards", [(k, o) for o in occs[:3] for k in range(n_rows - 1, -1, -1)]
    yield "every other row", [(k, o) for o in occs[:3] for k in range(0, n_rows, 2)]
    yield "one row again and again", [(1, occs[0])] * 9
    yield "no two alike", [(int(rng.integers(0, n_rows)), int(o)) for o in rng.choice(occs, 150)]
    yield "65 short runs", [(k, occs[r % len(occs)]) for r in range(65) for k in range(3)]


@pytest.mark.parametrize("ld_extra", [0, 1])
def test_runs(ld_extra):
    rng = np.random.default_rng(5)
    m = mixed_mir(0xA200, n_instr=500, reserved=True)
    n_rows = 37
    ld = m.n_occ + ld_extra
    host = rng.integers(0, 48, (n_rows, ld)).astype(np.uint16)
    rows = np.ascontiguousarray(host[:, :m.n_occ])
    dev = torch.from_numpy(host.view(np.int16)).cuda()
    an = vlo.analyze(m, interference=False, threads=8)
    hm, hl, _, _ = gpu_analyze([m], dense=False)
    try:
        occs = [int(o) for o in rng.integers(0, m.n_occ, 40)] + [0, m.n_occ - 1]
        for name, qs in orders(n_rows, occs, rng):
            masks = torch.full((len(qs), 16), -1, dtype=torch.int32, device="cuda")
            vl.vl_free_bases_multi([(hm[0], hl[0], dev[k], o) for k, o in qs], masks)
            torch.cuda.synchronize()
            got = masks.cpu().numpy().view(np.uint32)
            want = np.stack([vlo.free_bases(m, an, rows[k], o) for k, o in qs])
            bad = np.nonzero((got != want).any(axis=1))[0]
            assert len(bad) == 0, (name, [qs[j] for j in bad[:5]])
    finally:
        free(hm, hl)


@pytest.mark.parametrize("n_live,n_queries", [(255, 5), (256, 5), (257, 5), (600, 5), (40, 9000)])
def test_many_live_values_and_many_queries(n_live, n_queries):
    V = n_live + 1
    blocks = [[([v], []) for v in range(V)] + [([], list(range(v, min(V, v + 40)))) for v in range(0, V, 40)]]
    m = Mir.build(blocks, [[]], V, (512,), np.zeros(V, np.uint8), np.ones(V, np.uint8), np.ones(V, np.uint8), None, name=f"live{n_live}")
    rng = np.random.default_rng(n_live)
    rows = np.ascontiguousarray(rng.integers(0, 512, (7, V)).astype(np.uint16)[:, m.occ_vreg])
    an = vlo.analyze(m, interference=False)
    hm, hl, _, _ = gpu_analyze([m], dense=False)
    try:
        dev, ld = vl.rows_to_device(rows)
        qs = [(j % 7, n_live) for j in range(n_queries)]   # the last value's definition, all others live
        masks = torch.full((n_queries, 16), -1, dtype=torch.int32, device="cuda")
        rows_dev = [dev[k] for k in range(7)]
        vl.vl_free_bases_multi([(hm[0], hl[0], rows_dev[k], o) for k, o in qs], masks)
        torch.cuda.synchronize()
        got = masks.cpu().numpy().view(np.uint32)
        want = np.stack([vlo.free_bases(m, an, rows[k], n_live) for k in range(7)])
        assert (got == want[[k for k, _ in qs]]).all()
    finally:
        free(hm, hl)


@pytest.mark.parametrize("missing", ["mir", "live", "cand"])
def test_null_pointers_in_a_later_query(missing):
    k = gen.Kernel(gen.STRAIGHT, 3, 60, 60)
    hm = vl.vl_mir_create(k.mir)
    hl = vl.vl_liveness(hm)
    rows = torch.zeros((1, vl.pad_ld(k.mir.n_occ)), dtype=torch.int16, device="cuda")
    masks = torch.zeros((3, 16), dtype=torch.int32, device="cuda")
    try:
        queries = vl.make_mask_queries([(hm, hl, rows, 0)] * 3)
        setattr(queries[2], missing, None)
        with pytest.raises(vl.VlError) as e:
            vl.vl_free_bases_multi(queries, masks)
        assert e.value.code == -1
    finally:
        torch.cuda.synchronize()
        vl.vl_live_destroy(hl)
        vl.vl_mir_destroy(hm)


@pytest.mark.parametrize("n_live", [511, 512, 700])
@pytest.mark.parametrize("together", [1, 2])
def test_queries_that_stand_alone(n_live, together):
    """more runs than travel as an argument, of one query or two: first and later mentions, in P(i) as many
    values as are listed, one more and many more"""
    V = n_live + 1
    blocks = [[([v], []) for v in range(V)] + [([], list(range(v, min(V, v + 40)))) for v in range(0, V, 40)]]
    rng = np.random.default_rng(n_live + together)
    reserved = np.zeros((1, 16), np.uint32)
    reserved[0, 3] = 0xF0
    m = Mir.build(blocks, [[]], V, (512,), np.zeros(V, np.uint8), rng.choice([1, 2, 32], V, p=[0.8, 0.15, 0.05]), np.ones(V, np.uint8),
                  reserved, name=f"alone{n_live}")
    rows = np.ascontiguousarray(rng.integers(0, 640, (9, V)).astype(np.uint16)[:, m.occ_vreg])
    an = vlo.analyze(m, interference=False)
    hm, hl, _, _ = gpu_analyze([m], dense=False)
    try:
        dev, ld = vl.rows_to_device(rows)
        qs = [(0, n_live), (4, n_live)] + [(int(rng.integers(8)), int(o)) for o in rng.choice(m.n_occ, 150)]
        qs = [(k + t, o) for k, o in qs for t in range(together)]
        masks = torch.full((len(qs), 16), -1, dtype=torch.int32, device="cuda")
        vl.vl_free_bases_multi([(hm[0], hl[0], dev[k], o) for k, o in qs], masks)
        torch.cuda.synchronize()
        want = np.stack([vlo.free_bases(m, an, rows[k], o) for k, o in qs])
        assert (masks.cpu().numpy().view(np.uint32) == want).all()
    finally:
        free(hm, hl)


def test_more_runs_than_the_table_starts_with():
    """70,000 queries in no order, over and over from a few dozen different ones"""
    m = mixed_mir(0xA203, n_instr=200, reserved=True)
    rng = np.random.default_rng(8)
    rows = rng.integers(0, 48, (6, m.n_occ)).astype(np.uint16)
    an = vlo.analyze(m, interference=False, threads=8)
    pairs = [(int(rng.integers(6)), int(o)) for o in rng.integers(0, m.n_occ, 60)]
    want = np.stack([vlo.free_bases(m, an, rows[k], o) for k, o in pairs])
    which = rng.integers(0, len(pairs), 70000)
    hm, hl, _, _ = gpu_analyze([m], dense=False)
    try:
        dev, ld = vl.rows_to_device(rows)
        at = [dev[k] for k in range(6)]
        queries = vl.make_mask_queries([(hm[0], hl[0], at[pairs[w][0]], pairs[w][1]) for w in which])
        for _ in range(2):
            masks = torch.full((len(which), 16), -1, dtype=torch.int32, device="cuda")
            vl.vl_free_bases_multi(queries, masks)
            torch.cuda.synchronize()
            assert (masks.cpu().numpy().view(np.uint32) == want[which]).all()
    finally:
        free(hm, hl)


@pytest.mark.parametrize("n_live", [255, 256, 257, 510, 511, 512, 513, 767, 768, 769, 1100])
@pytest.mark.parametrize("tile_len", [100, 4096])
def test_lists_longer_than_a_thread_keeps(n_live, tile_len):
    """live-in lists around the 256 entries and tiles around the 768 events whose records stay in registers, and around the
    512 values that are listed from longer ones; half of the values are of another file, some are written twice"""
    rng = np.random.default_rng(n_live)
    V = n_live + 1
    vclass = (np.arange(V) % 2).astype(np.uint8)
    width = rng.choice([1, 1, 2, 4], V).astype(np.uint8)
    twice = [([int(v)], []) for v in rng.choice(n_live, 40)]
    blocks = [[([v], []) for v in range(n_live)] + twice + [([n_live], [])] + [([], list(range(v, min(V, v + 40)))) for v in range(0, V, 40)]]
    m = Mir.build(blocks, [[]], V, (512, 512), vclass, width, np.ones(V, np.uint8), None, name=f"live{n_live}")
    rows = rng.integers(0, 512, (9, m.n_occ)).astype(np.uint16)
    an = vlo.analyze(m, interference=False, threads=8)
    hm = [vl.vl_mir_create(m)]
    hl = vl.vl_liveness_multi(hm, tile_len=tile_len)
    try:
        dev, _ = vl.rows_to_device(rows)
        first = int(np.nonzero(m.occ_vreg == n_live)[0][0])
        qs = [(k, o) for o in (first, n_live // 2, first + 1) for k in range(len(rows))]
        masks = torch.full((len(qs), 16), -1, dtype=torch.int32, device="cuda")
        vl.vl_free_bases_multi([(hm[0], hl[0], dev[k], o) for k, o in qs], masks)
        torch.cuda.synchronize()
        got = masks.cpu().numpy().view(np.uint32)
        want = np.stack([vlo.free_bases(m, an, rows[k], o) for k, o in qs])
        assert (got == want).all()
    finally:
        free(hm, hl)


@pytest.mark.parametrize("n_values,times", [(30, 4), (60, 4), (255, 1), (256, 1), (257, 1), (300, 1)])
def test_values_with_many_records(n_values, times):
    """values that end and are written again within one tile: several records each, listed once; more of them than there is room
    for are found by their bits"""
    V = n_values + 1
    rng = np.random.default_rng(n_values + times)
    ins = [([v], []) for v in range(n_values)]
    for _ in range(times):
        for v in range(n_values):
            ins += [([], [v]), ([v], [])]
    ins += [([n_values], [])] + [([], list(range(v, min(V, v + 40)))) for v in range(0, V, 40)]
    m = Mir.build([ins], [[]], V, (512,), np.zeros(V, np.uint8), rng.choice([1, 1, 2], V), np.ones(V, np.uint8), None, name=f"again{n_values}")
    rows = rng.integers(0, 512, (9, m.n_occ)).astype(np.uint16)
    an = vlo.analyze(m, interference=False, threads=8)
    first = int(np.nonzero(m.occ_vreg == n_values)[0][0])
    want = np.stack([vlo.free_bases(m, an, rows[k], first) for k in range(len(rows))])
    hm = [vl.vl_mir_create(m)]
    try:
        dev, _ = vl.rows_to_device(rows)
        for tile_len in (512, 1024):   # at most 768 events, and more
            hl = vl.vl_liveness_multi(hm, tile_len=tile_len)
            masks = torch.full((len(rows), 16), -1, dtype=torch.int32, device="cuda")
            vl.vl_free_bases_multi([(hm[0], hl[0], dev[k], first) for k in range(len(rows))], masks)
            torch.cuda.synchronize()
            vl.vl_live_destroy(hl[0])
            assert (masks.cpu().numpy().view(np.uint32) == want).all(), tile_len
    finally:
        vl.vl_mir_destroy(hm[0])
