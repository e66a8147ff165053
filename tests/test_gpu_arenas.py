"""Analyses made and destroyed in turn, so that each finds the memory another one left: sizes up and
down, with and without dense points, from two threads with a stream each; against the oracle, exactly."""
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_2506_17506_amd as vl  # noqa: E402
from oracle import vlo  # noqa: E402
from vlgen import gen  # noqa: E402
from test_gpu_parity import assert_liveness_equal, assert_results_equal  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    vl.load()


def test_memory_of_earlier_analyses():
    work = []
    for n in (9000, 1500, 4000, 12000, 2500, 6000):   # analyses of some 1 to 25 MB
        k = gen.Kernel(gen.MHA, 31 + n, n, n * 3 // 4)
        rows, _ = k.candidates(n, 20, 8, 2)
        an = vlo.analyze(k.mir, threads=8)
        work.append((k.mir, rows, an, vlo.verify(k.mir, an, rows, threads=8)))
    errors = []

    def loop(order):
        try:
            stream = torch.cuda.Stream()
            with torch.cuda.stream(stream):
                for step, x in enumerate(order):
                    m, rows, an, want = work[x]
                    hm = vl.vl_mir_create(m)
                    hl = vl.vl_liveness_multi([hm], vl.VL_DENSE_POINTS if step % 3 == 0 else 0)[0]
                    dev, ld = vl.rows_to_device(rows)
                    stream.wait_stream(torch.cuda.default_stream())
                    out = torch.zeros((len(rows), 4), dtype=torch.int32, device="cuda")
                    vl.vl_verify_batch(hm, hl, dev, len(rows), ld, out)
                    stream.synchronize()
                    assert_results_equal(want, out.cpu().numpy().view(np.uint32).copy().view(vl.RESULT_DTYPE).reshape(-1), f"step {step}")
                    if step % 2:
                        assert_liveness_equal(m, an, vl.view_to_numpy(vl.vl_live_get(hl)), f"step {step}")
                    vl.vl_verify_batch(hm, hl, dev, len(rows), ld, out)   # still running when the memory is given back
                    vl.vl_live_destroy(hl)
                    vl.vl_mir_destroy(hm)
        except BaseException as e:   # noqa: BLE001
            errors.append(e)

    rng = np.random.default_rng(2)
    threads = [threading.Thread(target=loop, args=(rng.integers(0, len(work), 14).tolist(),)) for _ in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors[0]
