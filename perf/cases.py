"""The work whose speed counts: calls of the library as its users make them.

The library sits in a loop that samples register allocations for machine-IR kernels and
keeps the ones that verify.  What a program around it does, and what each path here stands for:

  verify    K samples of one or several kernels have come back from the model: the verdict of
            each (row-major, the layout of a stored batch, or occurrence-major, the layout a
            batched decoder leaves), then the loop's reductions (who passed, how many tries)
  step      analysis of every kernel into the handles it has, then verification of every
            candidate: the throughput benchmark's step
  analyse   the analysis alone, with the per-point live sets a caller can ask for
  arrive    kernels never seen before: create, analyse, verify, destroy; host data in hand
  count     every violation of every sample, by kind: the reward signal of a training run
  mask      the registers still free for the value a decoder is about to place: one decoding
            step (one query per sample of one kernel) or many kernels' steps at once
  bank      the register-bank conflict score of the samples
  lanes     programs whose instructions read parts of tuples: rows expanded to the rewritten
            program's numbering, then verified

Kernel shapes are the generator's: straight-line, a three-block loop, GEMM-shaped and
attention-shaped, at the sizes of the benchmark's configurations (200 / 2,000 / 8,000 / 20,000
instructions, and sweeps log-uniform in 1,000-20,000) with K = 64, 100 and 1,000 samples.
"""
import math
import os
import random
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import torch

import paper_2506_17506_amd as vl
from vlgen import gen

KIND = {"straight": gen.STRAIGHT, "loop": gen.LOOP3, "gemm": gen.GEMM, "mha": gen.MHA}
# what the generators produce: occurrences per instruction on average and at least, vregs per instruction, blocks
SHAPE = {"straight": (2.99, 2.9, 1.0, 1), "loop": (2.63, 2.45, 0.75, 3), "gemm": (2.87, 2.4, 0.75, 22),
         "mha": (2.84, 2.6, 0.75, 19), "sweep": (2.86, 2.4, 0.75, 20)}


def listed():
    def case(name, path, shape, n, kernels, k, **more):
        return {"name": name, "path": path, "shape": shape, "n": n, "kernels": kernels, "k": k, "damaged": 0.2, **more}
    return [
        # the smallest verification: 200 straight-line instructions, 64 samples, half of them damaged
        case("verify_straight200_k64", "verify", "straight", 200, 1, 64, damaged=0.5, layout="row"),
        # one mid-sized loop kernel analysed, dense live sets included
        case("analyse_loop2000_dense", "analyse", "loop", 2000, 1, 0, dense=True),
        # one GEMM-shaped kernel with many samples: analysis and verification
        case("step_gemm8000_k1000", "step", "gemm", 8000, 1, 1000, damaged=0.3, layout="row"),
        # the throughput benchmark: 256 kernels, 1,000-20,000 instructions, 100 samples each
        case("step_sweep256_k100", "step", "sweep", 20000, 256, 100, layout="row"),
        # one round of the regeneration loop over 64 large attention-shaped kernels, from the decoder's layout
        case("verify_mha64_k100_occ", "verify", "mha", 20000, 64, 100, layout="occ"),
        # what is left of a suite after the first tries: few samples, rows packed without padding
        case("verify_ragged24_k37", "verify", "sweep", 12000, 24, 37, layout="packed"),
        # a set of kernels that arrives with its first samples
        case("arrive_sweep16_k100", "arrive", "sweep", 16000, 16, 100, layout="row"),
        # all violations of a training batch
        case("count_sweep64_k100", "count", "sweep", 20000, 64, 100, layout="row"),
        # one decoding step of one kernel's 100 samples, and the same for many kernels in one call
        case("mask_mha5000_k100", "mask", "mha", 5000, 1, 100, layout="row"),
        case("mask_sweep64_k100", "mask", "sweep", 20000, 64, 100, layout="row"),
        # quality of one kernel's samples, four banks as in the paper's example
        case("bank_mha10000_k100", "bank", "mha", 10000, 1, 100, layout="row", banks=4),
        # one kernel whose operands read parts of tuples
        case("lanes_mha4000_k100", "lanes", "mha", 4000, 1, 100, layout="row"),
    ]


def draw(rng):
    """One more case of the ranges above; every size is drawn on a logarithmic scale."""
    def spread(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    path = rng.choice(["verify", "verify", "step", "step", "analyse", "arrive", "count", "mask", "bank", "lanes"])
    shape = rng.choice(["straight", "loop", "gemm", "mha", "sweep", "sweep"])
    n = {"straight": spread(60, 400), "loop": spread(200, 4000)}.get(shape) or spread(1000, 20000)
    kernels = 1 if path in ("bank", "lanes") else spread(1, {"arrive": 16, "count": 64, "analyse": 10}.get(path, 256))
    k = spread(1, 1000)
    if path == "lanes":
        n = min(n, 8000)
    if path == "analyse":
        n = min(n, 8000)   # the dense sets of ten kernels stay within a gigabyte
    # no more than the benchmark's 256 kernels of 6,200 instructions on average with 100 samples each
    mean = n if shape != "sweep" else (n - 1000) / math.log(n / 1000) if n > 1000 else n
    kernels = max(1, min(kernels, int(1.6e6 / mean)))
    k = max(1, min(k, 25600 // kernels, int({"count": 4e7, "arrive": 1e7, "bank": 1e7, "lanes": 1e6, "mask": 6e7}.get(path, 1.5e8) / (mean * kernels))))
    c = {"path": path, "shape": shape, "n": n, "kernels": kernels, "k": k, "damaged": round(rng.uniform(0.05, 0.5), 2),
         "layout": "row"}
    if path == "verify":
        c["layout"] = rng.choice(["row", "row", "occ", "packed"])
    elif path == "step":
        c["layout"] = rng.choice(["row", "packed"])
    elif path == "analyse":
        c.update(k=0, dense=rng.random() < 0.5)
    elif path == "bank":
        c["banks"] = rng.choice([2, 4, 4, 8])
    return c


def _sizes(case):
    """(kind, instructions) of every kernel; "sweep": the two large shapes in turn, sizes
    log-uniform from 1,000 to n (always one of them n)."""
    rng = random.Random(case["n"] * 1000 + case["kernels"])
    if case["shape"] != "sweep":
        return [(KIND[case["shape"]], case["n"])] * case["kernels"]
    hi = case["n"]
    out = []
    for i in range(case["kernels"]):
        n = hi if i == 0 else int(math.exp(rng.uniform(math.log(1000), math.log(hi)))) if hi > 1000 else hi
        out.append((gen.GEMM if i % 2 == 0 else gen.MHA, n))
    return out


def _make(kind, n, k, damaged, seed):
    """A kernel and its k samples (the generator's randomized first fit, a share of them damaged);
    a seed whose allocation fails is followed by another."""
    for bump in range(64):
        s = seed + (bump << 40)
        kern = gen.Kernel(kind, s, n, n if kind == gen.STRAIGHT else n * 3 // 4)
        if not k:
            return kern.mir, None
        try:
            rows, _ = kern.candidates(s ^ 0xC0FFEE, k, int(round(k * damaged)), {gen.STRAIGHT: 1, gen.GEMM: 3}.get(kind, 2))
        except RuntimeError:
            continue
        return kern.mir, rows
    raise RuntimeError("no allocation found")


class _Handles:
    """Programs and analyses; destroyed with the last object that refers to them."""

    def __init__(self):
        self.mirs, self.lives = [], []

    def __del__(self):
        for h in self.lives:
            vl.vl_live_destroy(h)
        for h in self.mirs:
            vl.vl_mir_destroy(h)


class _Array:
    """A device array of the library, for torch to look at.  The tensor keeps this object, and so
    the handles whose memory it shows."""

    def __init__(self, owner, ptr, shape, typestr):
        self.owner = owner
        self.__cuda_array_interface__ = {"data": (ptr, False), "shape": shape, "typestr": typestr, "version": 3}


def _look(owner, live, shape):
    """The results of one analysis as tensors over the library's memory.  Kill flags and interval
    runs: the part that every program of this shape and size has (nine tenths and more)."""
    v = vl.vl_live_get(live)
    w = v.words
    n_kill, n_run = int(SHAPE[shape][1] * v.n_instr), v.n_vreg
    assert n_kill <= v.n_occ and n_run <= v.n_seg
    shapes = {"live_in": (v.n_block, w), "live_out": (v.n_block, w), "occ_kill": (n_kill,), "seg_off": (v.n_vreg + 1,),
              "seg": (n_run, 2), "hull": (v.n_vreg, 2)}
    if v.live_after:
        shapes["live_after"] = (v.n_instr, w)
    return {name: torch.as_tensor(_Array(owner, getattr(v, name), shape, "|u1" if name == "occ_kill" else "<i4"), device="cuda")
            for name, shape in shapes.items()}


class State:
    """What a program around the library keeps: handles, device rows, job tables, result buffers."""

    def __init__(self):
        self.handles = _Handles()

    @property
    def mirs(self):
        return self.handles.mirs

    @property
    def lives(self):
        return self.handles.lives


def prepare(case, seed):
    vl.load()
    rng = random.Random(seed)
    path, k, layout = case["path"], case["k"], case.get("layout")
    sizes = _sizes(case)
    seeds = [rng.getrandbits(36) for _ in sizes]
    workers = min(16, os.cpu_count() or 1)
    with ThreadPoolExecutor(workers) as pool:
        made = list(pool.map(lambda a: _make(a[0][0], a[0][1], k, case["damaged"], a[1]), zip(sizes, seeds)))
    s = State()
    s.path, s.k, s.layout, s.n = path, k, layout, len(made)
    s.flags = vl.VL_DENSE_POINTS if case.get("dense") else 0
    s.host = [m for m, _ in made]
    s.rows, s.ld = [], []
    for m, rows in made:
        if rows is None:
            continue
        if layout == "packed":   # rows one after the other, no padding
            s.rows.append(torch.from_numpy(rows.view(np.int16)).cuda())
            s.ld.append(m.n_occ)
        elif layout == "occ":
            ld = (k + 7) // 8 * 8
            t = torch.zeros((m.n_occ, ld), dtype=torch.int16, device="cuda")
            t[:, :k] = torch.from_numpy(rows.view(np.int16)).cuda().t()
            s.rows.append(t)
            s.ld.append(ld)
        else:
            d, ld = vl.rows_to_device(rows)
            s.rows.append(d)
            s.ld.append(ld)
    del made
    if path in ("verify", "step", "arrive", "lanes"):
        s.out = torch.zeros((s.n * k, 4), dtype=torch.int32, device="cuda")
    if path == "count":
        s.out = torch.zeros((s.n * k, 8), dtype=torch.int32, device="cuda")
    if path == "arrive":
        return s
    if path == "lanes":
        # a quarter of the reads of pairs and quads take part of the tuple; writes are whole
        m, r = s.host[0], np.random.default_rng(seed)
        width = m.vreg_width[m.occ_vreg].astype(np.int64)
        part = (m.occ_flags == 2) & (width > 1) & (width <= 4) & (r.random(m.n_occ) < 0.25)
        lanes = np.where(part, r.integers(1, np.left_shift(1, width)), 0).astype(np.uint32)
        s.handles.mirs = [vl.vl_mir_create_lanes(m, lanes)]
        n_low = vl.vl_mir_lanes_get(s.mirs[0])["n_occ_low"]
        s.ld_low = vl.pad_ld(int(6.5 * m.n_instr))   # the most such a program becomes
        assert n_low <= s.ld_low
        s.low = torch.zeros((k, s.ld_low), dtype=torch.int16, device="cuda")
    else:
        s.handles.mirs = [vl.vl_mir_create(m) for m in s.host]
    if path == "bank":
        s.banks = case["banks"]
        s.out = torch.zeros(k, dtype=torch.int32, device="cuda")
        return s
    # the analysis every later call reads; a second one leaves the handles in the state a program's
    # repeated calls find them in
    s.handles.lives = vl.vl_liveness_multi(s.mirs, s.flags)
    if path in ("step", "analyse"):
        s.handles.lives = vl.vl_liveness_multi(s.mirs, s.flags, live=s.lives)
        # results stay where they are when handles are recycled: ten kernels' at most are returned
        s.views = [_look(s.handles, h, case["shape"]) for h in s.lives[:: max(1, -(-s.n // (8 if s.flags else 10)))]]
    if path in ("verify", "step"):
        s.jobs = vl.make_jobs([(m, l, d, k, ld, s.out[i * k:(i + 1) * k])
                               for i, (m, l, d, ld) in enumerate(zip(s.mirs, s.lives, s.rows, s.ld))])
        s.summaries = torch.zeros((s.n, 6), dtype=torch.int32, device="cuda")
        s.loop = torch.zeros(6, dtype=torch.int64, device="cuda")
    if path == "count":
        s.jobs = [(m, l, d, k, ld, s.out[i * k:(i + 1) * k])
                  for i, (m, l, d, ld) in enumerate(zip(s.mirs, s.lives, s.rows, s.ld))]
    if path == "mask":
        # every sample of a kernel is at the same occurrence: the first mention of some vreg
        queries = []
        for m, h, l, d in zip(s.host, s.mirs, s.lives, s.rows):
            firsts = np.unique(m.occ_vreg, return_index=True)[1]
            occ = int(firsts[rng.randrange(len(firsts))])
            queries += [(h, l, d[r], occ) for r in range(k)]
        s.queries = vl.make_mask_queries(queries)
        s.out = torch.zeros((len(queries), 16), dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    return s


def run(s):
    if s.path == "verify":
        if s.layout == "occ":
            vl.vl_verify_multi_occ_major(s.jobs)
        elif s.n == 1:
            vl.vl_verify_batch(s.mirs[0], s.lives[0], s.rows[0], s.k, s.ld[0], s.out)
        else:
            vl.vl_verify_multi(s.jobs)
        if s.n == 1:
            return s.out
        vl.vl_summarize_multi(s.jobs, s.summaries, s.loop)
        return s.out, s.summaries, s.loop
    if s.path == "step":
        vl.vl_liveness_multi(s.mirs, 0, live=s.lives)
        vl.vl_verify_multi(s.jobs)
        return s.out, s.views
    if s.path == "analyse":
        vl.vl_liveness_multi(s.mirs, s.flags, live=s.lives)
        return s.views
    if s.path == "arrive":
        mirs = [vl.vl_mir_create(m) for m in s.host]
        lives = vl.vl_liveness_multi(mirs)
        vl.vl_verify_multi([(m, l, d, s.k, ld, s.out[i * s.k:(i + 1) * s.k])
                            for i, (m, l, d, ld) in enumerate(zip(mirs, lives, s.rows, s.ld))])
        for h in lives:
            vl.vl_live_destroy(h)
        for h in mirs:
            vl.vl_mir_destroy(h)
        return s.out
    if s.path == "count":
        vl.vl_count_violations_multi(s.jobs)
        return s.out
    if s.path == "mask":
        vl.vl_free_bases_multi(s.queries, s.out)
        return s.out
    if s.path == "bank":
        vl.vl_bank_conflicts(s.mirs[0], s.rows[0], s.k, s.ld[0], s.banks, s.out)
        return s.out
    vl.vl_lanes_expand(s.mirs[0], s.rows[0], s.k, s.ld[0], s.low, s.ld_low)
    vl.vl_verify_batch(s.mirs[0], s.lives[0], s.low, s.k, s.ld_low, s.out)
    return s.low, s.out


def work(case):
    """Bytes one pass cannot do without, from the generators' usual proportions: the samples and the
    program read once, the results written once.  (Nothing here is a floating-point operation.)"""
    path, k = case["path"], case["k"]
    per, _, vper, blocks = SHAPE[case["shape"]]
    sizes = [n for _, n in _sizes(case)]
    total = 0.0
    for n in sizes:
        o, v = per * n, vper * n
        words = v / 32
        # program (vreg and flags of every occurrence, offsets, attributes); the analysis' results
        program = 5 * o + 4 * n + 3 * v
        analysis = o + 8 * blocks * words + 8 * v + 4 * v + 8 * v + (4 * n * words if case.get("dense") else 0)
        rows = k * 2 * o
        if path == "verify":
            total += rows + program + k * 16
        elif path in ("step", "arrive"):
            total += rows + program + analysis + k * 16
        elif path == "analyse":
            total += program + analysis
        elif path == "count":
            total += rows + program + 20 * v + k * 32
        elif path == "mask":
            # of the row only the registers of the values live at the query (some tens) are needed
            total += k * (64 + 32 + 2 * 64)
        elif path == "bank":
            total += rows + program + k * 4
        else:   # lanes: rows read, the expanded rows (about twice as long) written
            total += rows + 2 * rows + program + k * 16
    return {"bytes": total, "flops": 0.0}


def tolerance(case):
    return "exact"   # verdicts, counts, sets and intervals are whole numbers
