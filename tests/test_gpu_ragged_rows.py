"""Row-major samples of any pitch and alignment: every start within a word, programs that end anywhere in a
chunk, rows that end with the memory, and a pitch so large that a group of rows is cut to stay within 4 GB."""
import numpy as np
import pytest
import torch

import paper_2506_17506_amd as vl
from oracle import vlo
from vlgen import gen

pytestmark = pytest.mark.gpu


def _check(k, rows, dev, ld):
    an = vlo.analyze(k.mir)
    want = vlo.verify(k.mir, an, rows)
    hm = vl.vl_mir_create(k.mir)
    hl = vl.vl_liveness(hm)
    out = torch.zeros((rows.shape[0], 4), dtype=torch.int32, device="cuda")
    vl.vl_verify_batch(hm, hl, dev, rows.shape[0], ld, out)
    got = out.cpu().numpy().view(np.uint32).copy().view(vl.RESULT_DTYPE).reshape(-1)
    vl.vl_live_destroy(hl)
    vl.vl_mir_destroy(hm)
    assert set(want["status"]) >= {0, 1, 3}
    assert (got == want).all()


@pytest.mark.parametrize("shift", [0, 1, 2, 3])
@pytest.mark.parametrize("n_instr,pad", [(61, 0), (64, 1), (87, 2), (150, 3), (151, 4), (152, 5)])
def test_pitch_and_alignment(n_instr, pad, shift):
    k = gen.Kernel(gen.STRAIGHT, 4000 + n_instr, n_instr, n_instr)
    rows, _ = k.candidates(77 + n_instr, 70, 40, 1)
    ld = k.mir.n_occ + pad
    flat = np.full(shift + 69 * ld + k.mir.n_occ, 0xFFFF, np.uint16)   # ends with the last row
    for r in range(70):
        flat[shift + r * ld: shift + r * ld + k.mir.n_occ] = rows[r]
    dev = torch.from_numpy(flat.view(np.int16)).cuda()
    _check(k, rows, dev[shift:], ld)


@pytest.mark.parametrize("ld,n_rows", [((1 << 30) + 1, 4), ((1 << 26) + 8, 40)])
def test_pitch_beyond_32_bits(ld, n_rows):
    k = gen.Kernel(gen.STRAIGHT, 4999, 150, 150)
    rows, _ = k.candidates(5, n_rows, n_rows * 3 // 4, 1)
    n_occ = k.mir.n_occ
    dev = torch.empty((n_rows - 1) * ld + n_occ, dtype=torch.int16, device="cuda")
    for r in range(n_rows):
        dev[r * ld: r * ld + n_occ] = torch.from_numpy(rows[r].view(np.int16)).cuda()
    _check(k, rows, dev, ld)
