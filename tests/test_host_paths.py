"""The library's host code on a stand-in runtime: what it allocates, uploads and launches, and what it
does when memory runs out."""
import ctypes as C

import numpy as np

from stand_in import in_own_process
from vlgen.mir import Mir

S1 = 0x1000   # a stream, to the library a handle like any other


def program(n=8):
    return Mir.build([[((v,), ()) for v in range(n)] + [((), (v,)) for v in range(n)]], [[]], n, [64])


def analysed(s, how_many):
    hm = [s.vl.vl_mir_create(program(8 + k)) for k in range(how_many)]
    hl = s.vl.vl_liveness_multi(hm, stream=S1)
    return hm, hl


class Buffer:
    """host memory that stands for a device buffer"""
    def __init__(self, n_bytes):
        self.mem = np.zeros(n_bytes + 64, np.uint8)

    def data_ptr(self):
        return (self.mem.ctypes.data + 63) & ~63


def jobs_of(s, hm, hl, K, record=16):
    bufs = [(Buffer(K * 128), Buffer(K * record)) for _ in hm]
    return [(m, l, c, K, 64, o) for m, l, (c, o) in zip(hm, hl, bufs)], bufs


@in_own_process
def test_reductions_after_a_verification_that_ran_out_of_memory(s):
    """whichever allocation of the verification fails: the reductions that follow have their counter"""
    hm, hl = analysed(s, 2)
    jobs, keep = jobs_of(s, hm, hl, 8)
    arr = s.vl.make_jobs(jobs)
    sums, stats = Buffer(48), Buffer(48)
    failed = 0
    for stream, fail in ((S1, 0), (S1 + 1, 1)):   # a stream's first call allocates its table and its board
        s.fail_allocation(fail)
        try:
            s.vl.vl_verify_multi(arr, stream=stream)
        except s.vl.VlError as e:
            assert e.code == -6
            failed += 1
        s.launches.clear()
        s.vl.vl_summarize_multi(arr, sums, stats, stream=stream)
        (launch,) = [x for x in s.launches if "k_summarize" in x[0]]
        assert launch[5][1] != 0, "no counter"
    assert failed == 2
    # a board that was given up for a larger one that could not be had
    many, keep2 = jobs_of(s, hm, hl, 8)
    big = s.vl.make_jobs(many)
    for j in big:
        j.K = 1 << 20   # (nothing is read: the kernels are not run)
    s.vl.vl_verify_multi(arr, stream=S1)
    s.fail_allocation(0)
    try:
        s.vl.vl_verify_multi(big, stream=S1)
        raise AssertionError("the allocation did not fail")
    except s.vl.VlError as e:
        assert e.code == -6
    for which in (arr, big):
        s.launches.clear()
        s.vl.vl_summarize_multi(which, sums, stats, stream=S1)
        assert [x[5][1] != 0 for x in s.launches if "k_summarize" in x[0]] == [True]


@in_own_process
def test_counting_leaves_the_streams_verification_as_it_was(s):
    """a recorded verification replays over the table it was recorded with, and a loop of verifying and
    counting uploads nothing once it has settled"""
    hm, hl = analysed(s, 3)
    jobs, keep = jobs_of(s, hm, hl, 8)
    counts, keep2 = jobs_of(s, hm, hl, 8, record=32)
    arr = s.vl.make_jobs(jobs)
    s.vl.vl_verify_multi(arr, stream=S1)
    (table,) = [x[5][0] for x in s.launches if "k_walk" in x[0]]
    before = C.string_at(table, 3 * 32)
    for _ in range(9):   # more than there are workspaces and staged tables
        s.launches.clear()
        s.vl.vl_count_violations_multi(counts, stream=S1)
        assert [x[5][0] != table for x in s.launches if "k_walk" in x[0]] == [True]
        assert C.string_at(table, 3 * 32) == before
        uploads = s.counts()["uploads"]
        s.vl.vl_verify_multi(arr, stream=S1)
        assert s.counts()["uploads"] == uploads, "the table was uploaded again"


@in_own_process
def test_counting_takes_no_streams_place(s):
    """four streams verify without waiting for the device, whatever other streams count"""
    hm, hl = analysed(s, 2)
    jobs, keep = jobs_of(s, hm, hl, 8)
    counts, keep2 = jobs_of(s, hm, hl, 8, record=32)
    arr = s.vl.make_jobs(jobs)
    for k in range(8):
        s.vl.vl_count_violations_multi(counts, stream=S1 + 100 + k)
    for _ in range(2):
        for k in range(4):
            s.vl.vl_verify_multi(arr, stream=S1 + k)
            s.vl.vl_count_violations_multi(counts, stream=S1 + 200)
    assert s.counts()["device_waits"] == 0


@in_own_process
def test_reductions_over_more_samples_than_a_verification_takes(s):
    """no memory per sample is needed, so their number is bounded per job alone"""
    hm, hl = analysed(s, 1)
    jobs, keep = jobs_of(s, hm * 3, hl * 3, 8)
    arr = s.vl.make_jobs(jobs)
    for j in arr:
        j.K = 1 << 31   # (nothing is read: the kernels are not run)
    sums, stats = Buffer(72), Buffer(48)
    s.vl.vl_summarize_multi(arr, sums, stats, stream=S1)
    assert sum("k_summarize" in x[0] for x in s.launches) == 1
    assert s.counts()["largest"] < 64 << 20


@in_own_process
def test_kept_memory_is_given_back_when_memory_runs_short(s):
    """whichever allocation of whichever call finds no memory: what destroyed analyses left is returned first"""
    n = 20000
    large = s.vl.vl_mir_create(Mir.build([[((v,), ()) for v in range(n)] + [((), (v,)) for v in range(n)]], [[]], n, [64]))
    hm, hl = analysed(s, 2)

    def keep_some():
        for h in s.vl.vl_liveness_multi([large], stream=S1):
            s.vl.vl_live_destroy(h)

    def fails_once_and_recovers(what, after):
        keep_some()
        frees = s.counts()["frees"]
        s.fail_allocation(after)
        what()
        left = s.lib.stand_in_failing()
        s.fail_allocation(-1)
        if left:
            return False   # fewer allocations than that
        assert s.counts()["frees"] > frees
        return True

    made = []
    streams = iter(range(S1 + 1000, S1 + 2000))
    jobs, keep = jobs_of(s, hm, hl, 8)
    queries = s.vl.make_mask_queries([(hm[0], hl[0], keep[0][0], o % 8) for o in range(3000)])
    masks = Buffer(3000 * 64)

    def count():
        fresh, lives = analysed(s, 2)
        cj, k2 = jobs_of(s, fresh, lives, 8, record=32)
        s.vl.vl_count_violations_multi(cj, stream=S1)
    calls = {"create": lambda: made.append(s.vl.vl_mir_create(program())),
             "verify": lambda: s.vl.vl_verify_multi(jobs, stream=next(streams)),
             "count": count,
             "mask": lambda: s.vl.vl_free_bases_multi(queries, masks, stream=S1)}
    tried = {name: 0 for name in calls}
    for name, call in calls.items():
        while tried[name] < 20 and fails_once_and_recovers(call, tried[name]):
            tried[name] += 1
    assert tried["create"] >= 1 and tried["verify"] >= 2 and tried["count"] >= 8 and tried["mask"] >= 1, tried


@in_own_process
def test_block_sets_beyond_32_bit_indices(s):
    """few occurrences, but 2^32 words of block sets and more: cleared by the kernel that counts in 64 bits"""
    V = 32768
    for n_block, by_group in ((1 << 21, True), ((1 << 22) - 1, True), (1 << 22, False), ((1 << 22) + 5, False)):
        ins = np.zeros(n_block + 1, np.uint32)
        ins[1:] = 1   # the first block writes a value, the others are empty instructions
        m = Mir(np.arange(n_block + 1), np.r_[np.arange(n_block), n_block - 1], np.arange(1, n_block), ins, [0], [1],
                np.zeros(V, np.uint8), np.ones(V, np.uint8), np.ones(V, np.uint8), [64])
        hm = s.vl.vl_mir_create(m)
        s.launches.clear()
        hl = s.vl.vl_liveness_multi([hm], stream=S1)
        names = [x[0] for x in s.launches]
        assert any("k_group" in x for x in names) == by_group and any("k_zero" in x for x in names) != by_group
        s.vl.vl_live_destroy(hl[0])
        s.vl.vl_mir_destroy(hm)


@in_own_process
def test_boards_that_may_be_shared_are_left_zero(s):
    """the pair search writes the board's zeros for the entry point that allocates nothing, and for a stream's
    calls from the first that is recorded on: a pass of verification, or of reductions alone"""
    hm, hl = analysed(s, 2)
    jobs, keep = jobs_of(s, hm, hl, 8)
    arr, one = s.vl.make_jobs(jobs), s.vl.make_jobs(jobs[:1])
    sums, stats = Buffer(48), Buffer(48)
    s.lib.stand_in_record.argtypes = [C.c_void_p]

    def clears(call):
        s.launches.clear()
        call()
        (name,) = [x[0] for x in s.launches if "k_resolve" in x[0]]
        return "ELb1E" in name

    def verify(jobs_, stream):
        return clears(lambda: s.vl.vl_verify_multi(jobs_, stream=stream))
    m, l, cand, K, ld, out = jobs[0]
    assert clears(lambda: s.vl.vl_verify_batch_static(m, l, cand, K, ld, out, stream=S1))
    assert not verify(arr, S1) and not verify(one, S1) and not verify(arr, S1 + 1)
    s.lib.stand_in_record(S1)
    assert verify(arr, S1) and not verify(arr, S1 + 1)
    s.lib.stand_in_record(S1 + 1)
    s.vl.vl_summarize_multi(arr, sums, stats, stream=S1 + 1)
    s.lib.stand_in_record(None)
    assert verify(arr, S1) and verify(one, S1) and verify(arr, S1 + 1)
    assert verify(arr, 2) and not verify(arr, S1 + 2)   # 2: the thread's default stream


@in_own_process
def test_tables_of_runs_grow_with_the_runs(s):
    """many queries that fold into few runs take little memory, many that do not fold find room"""
    hm, hl = analysed(s, 2)
    rows, masks = Buffer(1 << 20), Buffer(64)
    base = rows.data_ptr()

    def query(occs):
        q = s.vl.make_mask_queries([(hm[0], hl[0], base + 128 * (j % 1000), int(o)) for j, o in enumerate(occs)])
        s.launches.clear()
        s.vl.vl_free_bases_multi(q, masks, stream=S1)
        (launch,) = [x for x in s.launches if "k_free_bases" in x[0]]
        return launch
    before = s.counts()["largest"]
    for _ in range(4):
        query(np.repeat(np.arange(100) % 8, 1000))   # 100 runs of 1,000
    assert s.counts()["largest"] <= max(before, 4096 * 48)
    for n in (4096, 4097, 20000):
        for _ in range(4):
            launch = query(np.arange(n) % 8)
            assert "alone" in launch[0] and launch[1][0] == n
    assert s.counts()["largest"] <= 65536 * 48


@in_own_process
def test_launches_of_many_tiles_stay_within_a_grid(s):
    """eight programs of four million instructions and a small one, tiles of one instruction: no launch has 2^32 threads in a row,
    dealt out to the dies or not"""
    n = 1 << 22
    off = np.zeros(n + 1, np.uint32)
    large = Mir([0, n], [0, 0], [], off, np.zeros(0, np.uint32), np.zeros(0, np.uint8), np.zeros(1, np.uint8), np.ones(1, np.uint8),
                np.ones(1, np.uint8), np.array([64], np.uint16))
    small = Mir([0, 1], [0, 0], [], off[:2], np.zeros(0, np.uint32), np.zeros(0, np.uint8), np.zeros(1, np.uint8), np.ones(1, np.uint8),
                np.ones(1, np.uint8), np.array([64], np.uint16))
    hm = [s.vl.vl_mir_create(large) for _ in range(8)] + [s.vl.vl_mir_create(small)]
    s.launches.clear()
    s.vl.vl_liveness_multi(hm, tile_len=1, stream=S1)
    assert any("k_stage_fill" in x[0] for x in s.launches)
    for name, grid, block, *_ in s.launches:
        assert grid[0] * block < 1 << 32 and grid[1] < 1 << 16, (name, grid, block)


@in_own_process
def test_queries_fold_into_runs_of_any_length(s):
    """the runs that travel with the launch, against a plain fold; lengths around those at which the queries are looked at eight at a time"""
    hm, hl = analysed(s, 2)
    masks = Buffer(64)
    seen = []
    plain = s.on_launch

    def on_launch(name, grid, block, lds, stream, args):
        if "k_free_bases" in name:
            n_runs = C.cast(args[1], C.POINTER(C.c_uint32))[0]
            seen.append(np.frombuffer(C.string_at(args[0], 48 * n_runs), np.int64).reshape(-1, 6).copy())
        plain(name, grid, block, lds, stream, args)
    s.on_launch = on_launch
    rng = np.random.default_rng(4)
    for length in [1, 2, 3, 8, 11, 12, 13, 14, 19, 20, 21, 22, 27, 28, 29, 30, 40]:
        queries, want = [], []   # (program, row, occurrence); (row, stride, occurrence, count)
        for j in range(12):
            which, row, step, occ = j % 2, 0x10000 + 0x1000 * j, [256, -512, 0][int(rng.integers(3))], int(rng.integers(8))
            queries += [(which, row + t * step, occ) for t in range(length)]
            want.append((row, step // 2 if length > 1 else 0, occ, length))
        if length > 1:   # ends that go on in all but one thing: the row, the occurrence, the program
            which, row, occ = queries[-1]
            step = queries[-1][1] - queries[-2][1]
            for q in ((which, row + step + 2, occ), (which, row + step + 4, (occ + 1) % 8), (1 - which, row + step + 6, (occ + 1) % 8)):
                queries.append(q)
                want.append((q[1], 0, q[2], 1))
        s.vl.vl_free_bases_multi(s.vl.make_mask_queries([(hm[w], hl[w], r, o) for w, r, o in queries]), masks, stream=S1)
        got = [(int(x[2]), int(x[3]), int(x[4] & 0xFFFFFFFF), int(x[4] >> 32)) for x in seen.pop()]
        assert got == want, (length, got, want)
