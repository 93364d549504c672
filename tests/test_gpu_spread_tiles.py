"""Single-call steps whose tile shrinks until the launch fills the chip (deposit
order, FP64, long FP32 sums): the same bits as the batch, whose tiles do not
shrink, and the oracle's outputs; sizes around the rule's 256 blocks."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import fd
from tests.gpu_util import to_dev, oracle_inputs, abs_bound, elementwise_ok, U32, U64

pytestmark = pytest.mark.gpu
cqc = pytest.importorskip("paper_2012_02333_amd")


@pytest.mark.parametrize("prec,out", [("fp32", torch.float32), ("fp64", torch.float64), ("fp32", torch.float64)])
@pytest.mark.parametrize("f,k,scattered", [((6, 8), 2, True), ((7, 11), 1, True), ((9, 11), 0, True), ((10, 12), 2, True),
                                           ((6, 8), 3, False), ((8, 11), 3, True), ((9, 10), 4, False)])
def test_spread_step(f, k, scattered, prec, out):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n = sum(f)
    order = np.random.default_rng(n + k).permutation(n) if scattered else np.arange(n)
    cut = W.CutMap(n, list(f), [0] * k, [1] * k, [int(q) for q in order])
    host, dev = to_dev(W.random_entries(cut, seed=1700 + k), torch.float64 if prec == "fp64" else torch.float32)
    c = cqc.CutMap.from_workload(cut)
    p, mass = cqc.reconstruct_fd(dev, c, precision=prec, out_dtype=out)
    xs = W.sample_outputs(n, 2048, seed=1701)
    e64 = oracle_inputs(host)
    got = p[torch.from_numpy(xs).cuda()].double().cpu().numpy()
    ok, info = elementwise_ok(got, fd.reconstruct(e64, cut, xs), abs_bound(e64, cut, xs), U32 if prec == "fp32" else U64,
                              4 ** k)
    assert ok, info
    assert abs(float(mass) - float(p.double().sum())) <= 1e-12 * float(p.double().abs().sum())
    if (prec == "fp64") == (out == torch.float64) and not (prec == "fp32" and k >= 3 and n >= 19):
        batch = cqc.Batch([dev, dev], [c, c], precision=prec)
        batch.run()
        assert torch.equal(batch.outs[0], p)
