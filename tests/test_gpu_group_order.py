"""Occurrences grouped by vreg and put in order, at the sizes where the work is cut: rounds of 1,024
and slices of 2,048 to 16,384 occurrences, values mentioned hundreds of times in a round (their group reaches
beyond what a workgroup has at hand), more than 2^17 occurrences or more vregs than LDS counts
(the large-program sort); the whole analysis and some verdicts against the oracle, exactly."""
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


def program(seed, n_occ, V, heavy, share):
    """n_occ occurrences: V values written once each, then reads of three at a time (every tenth
    instruction reads one value three times); `share` of the reads go to `heavy` of the values"""
    rng = np.random.default_rng(seed)
    n_read = n_occ - V
    reads = np.where(rng.random(n_read) < share, rng.integers(0, max(1, heavy), n_read), rng.integers(0, V, n_read))
    for k in range(0, n_read - 2, 30):
        reads[k:k + 3] = reads[k]
    occ_v = np.concatenate([rng.permutation(V), reads]).astype(np.uint32)
    occ_f = np.concatenate([np.full(V, 1), np.full(n_read, 2)]).astype(np.uint8)
    off = np.concatenate([np.arange(V + 1), V + np.minimum(n_read, np.arange(3, n_read + 3, 3))]).astype(np.uint32)
    off = off[:V + 1 + (n_read + 2) // 3]
    N = len(off) - 1
    cut = max(1, N // 3)
    blocks = ([0, cut, N], [0, 1, 1], [1]) if N > 1 else ([0, N], [0, 0], [])
    return Mir(*blocks, off, occ_v, occ_f, np.zeros(V, np.uint8),
               np.ones(V, np.uint8), np.ones(V, np.uint8), [512], None, name=f"occ{n_occ}_v{V}_h{heavy}")


CASES = [(1, 1, 0, 0.0), (1023, 40, 1, 0.9), (1024, 40, 2, 0.9), (1025, 300, 1, 0.5), (2047, 64, 1, 1.0), (5000, 2000, 3, 0.2),
         (16383, 900, 2, 0.6), (16384, 900, 1, 0.95), (16385, 5000, 4, 0.3), (40000, 300, 5, 0.8)]


@pytest.mark.parametrize("n_occ,V,heavy,share", CASES)
def test_rounds_and_slices(n_occ, V, heavy, share):
    m = program(n_occ, n_occ, V, heavy, share)
    an = vlo.analyze(m, threads=8)
    assert an.contract == 0
    hm, hl, got, _ = gpu_analyze([m])
    try:
        assert_liveness_equal(m, an, got[0], m.name)
        rng = np.random.default_rng(9)
        rows = np.zeros((5, n_occ), np.uint16)
        rows[:] = rng.integers(0, 512, (5, V))[:, m.occ_vreg]
        rows[1, rng.integers(0, n_occ, 3)] ^= 1
        assert_results_equal(vlo.verify(m, an, rows, threads=8), gpu_verify(hm, hl, [rows])[0], m.name)
    finally:
        free(hm, hl)


@pytest.mark.parametrize("n_occ,V,heavy,share", [(2048, 60, 2, 0.5), (2049, 700, 1, 0.9), (4097, 64, 3, 0.5), (16385, 300, 1, 1.0),
                                                 (65535, 6, 1, 1.0), (65536, 6, 1, 1.0), (65535, 9000, 5, 0.4)])
def test_slices_of_few_programs(n_occ, V, heavy, share):
    """slices of 2,048 and more, counts in half a word up to 65,535 occurrences (nearly all of one value)"""
    test_rounds_and_slices(n_occ, V, heavy, share)


@pytest.mark.parametrize("n_occ,V", [(140000, 200), (60000, 33000)])
def test_large_programs(n_occ, V):
    check_large_program(program(n_occ, n_occ, V, 3, 0.3))


@pytest.mark.parametrize("n_occ,V,share", [(40000, 32769, 0.5), (70000, 45000, 0.9), (150000, 100000, 1.0)])
def test_values_that_share_a_place(n_occ, V, share):
    """more vregs than LDS has counters for: the values mentioned again and again fall on one place of the slices' tables of
    8,192, and only one of them has it"""
    m = program(n_occ, n_occ, V, 4, share)
    name = np.arange(V, dtype=np.uint32)
    for k in range(4):
        name[[k, 7 + 8192 * k]] = name[[7 + 8192 * k, k]]
    m.occ_vreg = name[m.occ_vreg]
    check_large_program(m)


def check_large_program(m):
    V = m.n_vreg
    an = vlo.analyze(m, interference=False, threads=8) if V < 1000 else None
    hm, hl, got, _ = gpu_analyze([m], dense=V < 1000)
    try:
        g = got[0]
        if an is not None:
            assert_liveness_equal(m, an, g, m.name)
        # one run per value, from its definition to its last read (or past its definition)
        first = np.full(V, m.n_occ, np.int64)
        np.minimum.at(first, m.occ_vreg, np.arange(m.n_occ))
        last = np.zeros(V, np.int64)
        np.maximum.at(last, m.occ_vreg, np.arange(m.n_occ))
        instr = np.repeat(np.arange(m.n_instr), np.diff(m.instr_occ_off.astype(np.int64)))
        want = np.stack([instr[first], np.maximum(instr[last], instr[first] + 1)], axis=1)
        assert (g["seg_off"] == np.arange(V + 1)).all() and (g["seg"] == want).all() and (g["hull"] == want).all()
    finally:
        free(hm, hl)
