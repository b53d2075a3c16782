"""The batch's marching kernel through its call sequence: single steps only,
an aligning step on the other buffer set, replays of the captured graph with
passes and single steps after them.  (4, 16, 1, 16) is the marching kernel of
the rows and columns for which the default values stand for the tiles."""
import numpy as np
import pytest

from paper_2405_00814_amd import workloads as W

from helpers import assert_parity, rel_l2, run_gpu, run_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cfg", [(4, 16, 1, 16), (4, 8, 2, 0), (2, 16, 4, 0), (1, 16, 1, 0)])
def test_batch_marching_sequence(cfg):
    from paper_2405_00814_amd.sim import Batch
    probs = W.batch2d(count=5, steps=0, seed=3, side=(70, 190), nprobes=3, rect_side=(8, 40), rect_density=40.0 / 4096)
    b = Batch(probs)
    b.set_kernel(*cfg)
    b.step(3)
    launches = b.last_step_time()[1]
    b.step(34)
    b.step(150)
    assert b.last_step_time()[1] > launches
    for q, pb in enumerate(probs):
        got = {k: b.get_field(q, k) for k in ("ez", "hx", "hy")}
        single, srec, _ = run_gpu(pb, 187)
        for k in got:
            assert rel_l2(got[k], single[k]) <= 1e-5, (q, k)
        assert rel_l2(b.probe(q), srec) <= 1e-5
        ref, rrec = run_oracle(pb, 187)
        assert_parity(got, ref, 1e-4, "batch[%d]" % q)
        assert rel_l2(b.probe(q), rrec) <= 1e-4
    b.close()
