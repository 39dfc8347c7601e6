"""Batches of programs whose plans have narrower tiles than their states: explicit
plans of 12-qubit (and smaller) states on fewer bits, which the persistent kernel
cannot hold whole, and of 13 qubits on 4 and 3 bits, against the oracle, beside
programs planned by default. And the prefixes of streamed requests as items of a
persistent launch, where an arena has no room for the tables of their rounds."""
import numpy as np
import pytest

import workloads as W
from oracle import sim

pytestmark = pytest.mark.gpu


def test_narrow_plans_match_oracle():
    from paper_2604_11599_amd import Context
    ctx = Context(0)
    try:
        reqs, srcs = [], []
        for k, (n, tile_bits) in enumerate([(12, 11), (12, 10), (11, 10), (5, 4), (3, 2), (13, 4), (13, 3), (12, 12)]):
            src = W.random_dynamic_program(700 + k, n, n_ops=40, final_measure=True)
            p = ctx.load(src)
            p.replan(tile_bits, min(4, tile_bits), 0.5)
            srcs.append(src)
            reqs.append({"prog": p, "shots": 4, "seed": 30 + k})
        for k, (src, r) in enumerate(zip(srcs, ctx.run_batch(reqs))):
            for s in range(4):
                o = sim.run_shot(src, seed=30 + k, shot=s)
                if any(abs(e[3] - e[4]) < 1e-12 for e in o.events):
                    continue
                assert list(r.bits()[s]) == o.cbits, (k, s)
                assert abs(r.record_prob[s] - o.record_prob) < 1e-12
    finally:
        ctx.close()


def test_prefixes_without_room_for_their_tables():
    import torch
    from paper_2604_11599_amd import Context, QsvError
    srcs = [W.c3_program(3, n=14, layers=3), W.c3_program(4, n=13, layers=2)]
    ref = Context(0)
    buf = torch.empty(64 << 20, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()

    def run(ctx):
        return ctx.run_batch([{"prog": ctx.load(s), "shots": 5, "seed": 50 + k} for k, s in enumerate(srcs)])

    def run_in(size):
        ar = Context(0, arena=buf.data_ptr(), arena_bytes=size)
        try:
            return run(ar)
        except QsvError:
            return None
        finally:
            ar.close()

    try:
        want = run(ref)
        lo, hi = 0, buf.numel()  # the smallest arena that does: without the tables
        while hi - lo > 256:
            mid = (lo + hi) // 512 * 256
            lo, hi = (lo, mid) if run_in(mid) is not None else (mid, hi)
        for size in (hi, hi + 256, hi + 4096, buf.numel()):
            for a, b in zip(run_in(size), want):
                for x, y in [(a.creg, b.creg), (a.record, b.record), (a.record_prob, b.record_prob)]:
                    assert np.array_equal(x, y)
    finally:
        ref.close()
        del buf
