"""Calls that overlap although they share memory (the entry point that allocates nothing, called on two
streams; a recorded pass replayed on another stream than the one it was recorded on) have undefined
results, but the next ones are right again.  What overlaps here checks the same program on both sides,
cut into different numbers of tiles, so that whatever mixes stays a position of that program."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_2506_17506_amd as vl  # noqa: E402
from oracle import vlo  # noqa: E402
from vlgen import gen  # noqa: E402
from test_gpu_parity import assert_results_equal  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    vl.load()


def results(out):
    return out.cpu().numpy().view(np.uint32).reshape(-1, 4).copy().view(vl.RESULT_DTYPE).reshape(-1)


def test_overlapping_calls_spoil_no_later_one():
    k = gen.Kernel(gen.MHA, 0x0E0, 3000, 2250)
    rows, _ = k.candidates(3, 640, 300, 2)
    want = vlo.verify(k.mir, vlo.analyze(k.mir, threads=8), rows, threads=8)
    K = rows.shape[0]
    hm = vl.vl_mir_create(k.mir)
    fine, coarse = vl.vl_liveness_multi([hm], 0, 32), vl.vl_liveness_multi([hm], 0, 128)
    dev, ld = vl.rows_to_device(rows)
    outs = [torch.zeros((K, 4), dtype=torch.int32, device="cuda") for _ in range(2)]
    streams = [torch.cuda.Stream() for _ in range(2)]
    torch.cuda.synchronize()
    try:
        for _ in range(20):
            for live, out, stream in zip((fine, coarse), outs, streams):
                vl.vl_verify_batch_static(hm, live[0], dev, K, ld, out, stream=stream)
        torch.cuda.synchronize()
        for live in (coarse, fine):
            for o in outs:
                o.fill_(-1)
            vl.vl_verify_batch_static(hm, live[0], dev, K, ld, outs[0])
            torch.cuda.synchronize()
            assert_results_equal(want, results(outs[0]), "after the calls that overlapped")
    finally:
        torch.cuda.synchronize()
        for h in fine + coarse:
            vl.vl_live_destroy(h)
        vl.vl_mir_destroy(hm)


def test_overlapping_replays_spoil_no_later_pass():
    n = 12
    k = gen.Kernel(gen.MHA, 0x0E1, 3000, 2250)
    rows, _ = k.candidates(3, 120, 60, 2)
    want = vlo.verify(k.mir, vlo.analyze(k.mir, threads=8), rows, threads=8)
    K = rows.shape[0]
    hm = vl.vl_mir_create(k.mir)
    dev, ld = vl.rows_to_device(rows)
    side, other = torch.cuda.Stream(), torch.cuda.Stream()
    lives = []
    try:
        with torch.cuda.stream(side):
            passes = []
            for tile_len in (32, 128):
                live = vl.vl_liveness_multi([hm], 0, tile_len)
                lives += live
                outs = torch.zeros((n, K, 4), dtype=torch.int32, device="cuda")
                jobs = vl.make_jobs([(hm, live[0], dev, K, ld, outs[j]) for j in range(n)])
                sums = torch.zeros((n, 6), dtype=torch.int32, device="cuda")
                stats = torch.zeros(6, dtype=torch.int64, device="cuda")
                passes.append((jobs, outs, sums, stats))

            def run(p):
                vl.vl_verify_multi(p[0])
                vl.vl_summarize_multi(p[0], p[2], p[3])
            for p in passes:
                run(p)
            side.synchronize()
            run(passes[0])
            side.synchronize()
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=side):
                run(passes[0])
            single = vl.make_jobs([(hm, lives[1], dev, K, ld, passes[1][1][0])])
            for _ in range(20):
                with torch.cuda.stream(other):
                    graph.replay()
                vl.vl_verify_multi(single)   # one job: the recorded pass keeps its table
                vl.vl_summarize_multi(passes[0][0], passes[1][2], passes[1][3])
            torch.cuda.synchronize()
            hist = np.bincount(want["status"], minlength=4)
            for eager in (True, False):
                p = passes[0]
                for t in p[1:]:
                    t.fill_(-1)
                side.synchronize()
                run(p) if eager else graph.replay()
                torch.cuda.synchronize()
                for j in range(n):
                    assert_results_equal(want, results(p[1][j]), f"job {j}, {'eager' if eager else 'replay'}")
                s = p[3].cpu().numpy().view(np.uint64)
                assert (s[2:] == n * hist).all()
    finally:
        torch.cuda.synchronize()
        for h in lives:
            vl.vl_live_destroy(h)
        vl.vl_mir_destroy(hm)
