"""Split-BF16 chains whose intermediate is written as the bfloat16 parts of the
step that reads it: as that step's X and its Y operand, two-column rows, tiles
that overhang and whole ones, two and three parts, a further intermediate, the
scattered output order, dead rows, and a consumer that is no split step (the
FP32 intermediate).  Elementwise bound as in test_gpu_bf16x3; the batch, which
splits the FP32 intermediate while staging, gives the same outputs bit for bit."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import fd
from tests.gpu_util import to_dev, oracle_inputs, abs_bound, elementwise_ok, sum_terms, U32

pytestmark = pytest.mark.gpu
cqc = pytest.importorskip("paper_2012_02333_amd")


@pytest.mark.parametrize("prec", ["bf16x6", "bf16x3"])
@pytest.mark.parametrize("f,cuts,scattered", [
    ([3, 1, 5], [3, 3], False), ([5, 1, 3], [3, 3], False), ([5, 3, 1], [3, 3], False), ([2, 2, 6], [3, 4], True),
    ([3, 1, 2, 5], [3, 3, 3], False), ([4, 4, 6], [3, 2], False), ([7, 7, 7], [3, 3], False), ([8, 7, 8], [4, 3], True)])
def test_intermediate_in_parts(f, cuts, scattered, prec):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n, K = sum(f), sum(cuts)
    up = [c for c, k in enumerate(cuts) for _ in range(k)]
    order = list(np.random.default_rng(3).permutation(n)) if scattered else list(range(n))
    cut = W.CutMap(n, f, up, [u + 1 for u in up], [int(q) for q in order])
    zr = [(1, r) for r in range(cut.entry_shape(1)[0]) if r % 5 == 1]
    host, dev = to_dev(W.random_entries(cut, seed=1600, zero_rows=zr), torch.float32)
    c = cqc.CutMap.from_workload(cut)
    p, mass = cqc.reconstruct_fd(dev, c, precision=prec)
    xs = W.sample_outputs(n, 2048, seed=1601) if n > 14 else np.arange(2 ** n)
    e64 = oracle_inputs(host)
    terms = max(4 ** max(cuts), int(round(cqc.cost(c)[1] / 2 ** n)))
    got = p[torch.from_numpy(np.asarray(xs)).cuda()].double().cpu().numpy()
    ok, info = elementwise_ok(got, fd.reconstruct(e64, cut, xs), abs_bound(e64, cut, xs), U32, sum_terms(prec, terms))
    assert ok, info
    assert abs(float(mass) - float(p.double().sum())) <= 1e-12 * float(p.double().abs().sum())
    batch = cqc.Batch([dev, dev], [c, c], precision=prec)
    batch.run()
    assert torch.equal(batch.outs[0], p) and torch.equal(batch.outs[1], p)
