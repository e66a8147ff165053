"""All-violations counts where the work is cut: 0 to 9 failed samples (units of four), programs
whose pairs fill several parts, row pitches that allow 16-byte reads or not, a program with more
vregs than the table in LDS holds (19,456); against the oracle, exactly."""
import ctypes as C

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_2506_17506_amd as vl  # noqa: E402
from oracle import vlo  # noqa: E402
from vlgen import gen  # noqa: E402
from vlgen.mixed import mixed_mir  # noqa: E402
from test_gpu_parity import free, gpu_analyze  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    vl.load()


def compare(m, row_sets, pitches=(0,)):
    an = vlo.analyze(m, threads=8)
    hm, hl, _, _ = gpu_analyze([m], dense=False)
    try:
        for rows in row_sets:
            want = vlo.count_violations(m, an, rows, threads=8)
            K = rows.shape[0]
            for extra in pitches:
                ld = (m.n_occ + 7) // 8 * 8 + extra
                host = np.zeros((K, ld), np.uint16)
                host[:, :m.n_occ] = rows
                dev = torch.from_numpy(host.view(np.int16)).cuda()
                out = torch.full((K, 8), -1, dtype=torch.int32, device="cuda")
                for _ in range(2):
                    vl.vl_count_violations_multi([(hm[0], hl[0], dev, K, ld, out)])
                torch.cuda.synchronize()
                got = out.cpu().numpy().view(np.uint32)
                for c, name in enumerate(("kinds", "n_cons", "n_real", "n_safe", "real_bits")):
                    assert (got[:, c] == want[name]).all(), (m.name, K, extra, name)
    finally:
        free(hm, hl)


def test_failed_samples_and_parts():
    k = gen.Kernel(gen.MHA, 0xC0DE, 3001, 2250)
    rows, log = k.candidates(77, 24, 12, 2)
    good, bad = rows[log["kind"] == 0], rows[log["kind"] != 0]
    assert len(good) == 12 and len(bad) == 12
    rng = np.random.default_rng(3)
    wild = rng.integers(0, 600, (9, k.mir.n_occ)).astype(np.uint16)   # everything wrong at once
    sets = [np.ascontiguousarray(np.concatenate([good[:3], bad[:n]])) for n in (0, 1, 3, 4, 5, 8, 9)] + [good[:1], bad[:1], wild]
    compare(k.mir, sets, pitches=(0, 1, 8))


def test_mixed_shapes():
    m = mixed_mir(0xC300, n_instr=900, reserved=True)
    rng = np.random.default_rng(4)
    compare(m, [rng.integers(0, 64, (70, m.n_occ)).astype(np.uint16)], pitches=(0, 3))


def test_more_vregs_than_lds():
    k = gen.Kernel(gen.STRAIGHT, 0xC0DF, 20000, 20000)
    rows, _ = k.candidates(5, 6, 4, 1)
    compare(k.mir, [rows])


@pytest.mark.parametrize("n_instr", [61, 64, 200])
@pytest.mark.parametrize("K", [1, 70])
def test_rows_that_end_with_their_memory(n_instr, K):
    """nothing is asked of a row beyond its registers: the last one ends where the allocation does (the
    16 bytes, or the word, its last register lies in), whatever the pitch"""
    k = gen.Kernel(gen.STRAIGHT, 0xC0E0 + n_instr, n_instr, n_instr)
    m = k.mir
    rows, _ = k.candidates(9, K, K // 2, 1)
    an = vlo.analyze(m, threads=8)
    want = vlo.count_violations(m, an, rows, threads=8)
    hip = vl.binding.hip_runtime()
    size = 4 << 20
    mem = C.c_void_p()
    assert hip.hipMalloc(C.byref(mem), C.c_size_t(size)) == 0
    hm, hl, _, _ = gpu_analyze([m], dense=False)
    try:
        for ld, unit in ((vl.pad_ld(m.n_occ), 16), ((m.n_occ + 7) // 8 * 8, 16), (m.n_occ | 1, 4), (m.n_occ + 1 & ~1, 4)):
            used = (K - 1) * ld * 2 + m.n_occ * 2
            start = (size - used) // unit * unit
            host = np.zeros((size - start) // 2, np.uint16)
            for r in range(K):
                host[r * ld:r * ld + m.n_occ] = rows[r]
            assert hip.hipMemcpy(C.c_void_p(mem.value + start), host.ctypes.data_as(C.c_void_p), C.c_size_t(host.nbytes), 1) == 0
            out = torch.full((K, 8), -1, dtype=torch.int32, device="cuda")
            vl.vl_count_violations_multi([(hm[0], hl[0], mem.value + start, K, ld, out)])
            torch.cuda.synchronize()
            got = out.cpu().numpy().view(np.uint32)
            for c, name in enumerate(("kinds", "n_cons", "n_real", "n_safe", "real_bits")):
                assert (got[:, c] == want[name]).all(), (ld, name)
    finally:
        free(hm, hl)
        assert hip.hipFree(mem) == 0


def test_tables_of_every_kind_in_one_call():
    """programs whose registers fit LDS for four samples, for two, and not at all; nearly every sample, one
    of them and none failing, so that the pairs are cut into few parts and into many"""
    sets = []
    for j, (n, seed) in enumerate(((300, 1), (20000, 2), (39500, 3), (5000, 4))):
        k = gen.Kernel(gen.STRAIGHT, 0xC0F0 + seed, n, n)
        rows, log = k.candidates(5, 11, 9, 1)
        rows[9] = np.random.default_rng(j).integers(0, 512, k.mir.n_occ)
        sets.append((k.mir, rows, log["kind"] == 0))
    assert [m.n_vreg > x for (m, _, _), x in zip(sets[1:3], (19456, 38912))] == [True, True]
    ans = [vlo.analyze(m, threads=8) for m, _, _ in sets]
    hm, hl, _, _ = gpu_analyze([m for m, _, _ in sets], dense=False)
    try:
        for pick in (lambda good, n: np.arange(n), lambda good, n: np.r_[np.nonzero(good)[0], 0], lambda good, n: np.nonzero(good)[0]):
            jobs, wants = [], []
            for m, l, (mir, rows, good), an in zip(hm, hl, sets, ans):
                rows = np.ascontiguousarray(rows[pick(good, len(rows))])
                dev, ld = vl.rows_to_device(rows)
                out = torch.full((len(rows), 8), -1, dtype=torch.int32, device="cuda")
                jobs.append((m, l, dev, len(rows), ld, out))
                wants.append(vlo.count_violations(mir, an, rows, threads=8))
            for order in (jobs, jobs[::-1], jobs[1:2], jobs[2:3]):
                for j in order:
                    j[5].fill_(-1)
                vl.vl_count_violations_multi(order)
                torch.cuda.synchronize()
                for j, want in zip(jobs, wants):
                    if not any(j is x for x in order):
                        continue
                    got = j[5].cpu().numpy().view(np.uint32)
                    for c, name in enumerate(("kinds", "n_cons", "n_real", "n_safe", "real_bits")):
                        assert (got[:, c] == want[name]).all(), name
    finally:
        free(hm, hl)
