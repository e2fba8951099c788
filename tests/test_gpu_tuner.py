"""The fused batch's autotuner where candidates come to the same launches: disks of at most 32 rows, which any chunk length from
32 up sweeps as one chunk or, where that leaves the device idle, as the same shorter ones.  Nothing is to choose, and the
first candidate is kept, in whatever order they are given."""
import numpy as np
import pytest

from paper_1602_02359_amd import workloads as W

pytestmark = pytest.mark.gpu


def _solvers(precision, count=9, seed=8):
    from paper_1602_02359_amd import fargo as F
    out = []
    for p in W.disk_batch(count=count, nr_range=(8, 32), seed=seed):
        s = F.Solver(dict(p.params, precision=precision))
        s.upload(p.fields)
        out.append(s)
    return out


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_first_of_equal_candidates_is_kept(precision):
    from paper_1602_02359_amd import fargo as F
    for chunks in ((64, 32, 33, 40, 48, 56, 63, 96), (32, 96, 64, 33, 40, 48, 56, 63), (48, 32, 33, 40, 56, 63, 64, 96)):
        print("tuner", precision, chunks, flush=True)
        b = F.Batch(_solvers(precision), lanes=0)
        best = b.fargo_batch_tune(lanes=(0,), chunks=chunks, steps=1)
        assert best[1] == chunks[0] and list(b.chunks()) == [chunks[0]] * 9
        del b


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_a_class_keeps_its_chunk_beside_other_classes(precision):
    """Size classes tuned to different lengths: every disk still takes its own step, bit for bit."""
    import torch
    from paper_1602_02359_amd import fargo as F
    batch, own = _solvers(precision, 40, 9), _solvers(precision, 40, 9)
    b = F.Batch(batch, lanes=0)
    for chunks in ((3, 64, 5, 1), (1, 2, 7, 19)):
        b.fargo_batch_tune(lanes=(0,), chunks=chunks, steps=1)
        assert all(c in chunks for c in b.chunks())
        b.fargo_batch_step()
        for s in own:
            s.fargo_step(0.0)
        torch.cuda.synchronize()
        for s, o in zip(batch, own):
            for k in ("rho", "vx", "vy"):
                n = s.params["nx"]
                assert torch.equal(s.state[k][..., :n], o.state[k][..., :n])
    del b
