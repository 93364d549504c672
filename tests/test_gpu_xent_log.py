"""The FP32 loss logarithm where its relative accuracy is hardest: every output
near 1 (within 2^-1 to 2^-23 of it, both sides), and at the floor.  The loss of
a batch with a single target entry is one term, -t log max(p, 1e-30): an FP32
logarithm of at most 2 ulp leaves 2^-22 of it, whatever p."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu
cqc = pytest.importorskip("paper_2012_02333_amd")


@pytest.mark.parametrize("f,k", [((7, 8), 1), ((4, 5), 1), ((8, 6), 0)])
def test_loss_terms_near_one(f, k):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n = sum(f)
    cut = cqc.CutMap.from_workload(W.CutMap(n, list(f), [0] * k, [1] * k, list(range(n))))
    # X: one in the first row (2^k in all), Y: the values, so that p_x = y exactly
    vals = [1 + s * 2.0 ** -e for e in range(1, 24) for s in (1, -1)] + [1.0, 2.0, 1e-30, 1e-38, 0.0, 1e-10]
    y = np.resize(np.array(vals, dtype=np.float32), 2 ** f[1])
    ents = []
    for c, size in enumerate(f):
        E = np.zeros((4 ** k, 2 ** size), dtype=np.float32)
        E[0] = 2.0 ** k if c == 0 else y
        ents.append(torch.from_numpy(E).cuda())
    cases = list(range(min(len(vals), 2 ** f[1])))
    targets = []
    for j in cases:
        t = torch.zeros(2 ** n, device="cuda")
        t[j] = 0.75
        targets.append(t)
    batch = cqc.Batch([ents] * len(cases), [cut] * len(cases), precision="fp32", targets=targets, with_loss=True)
    batch.run()
    got = batch.losses.cpu().numpy()
    for j in cases:
        p = float(batch.outs[j][j])
        assert p == float(y[j]), (j, p)
        want = -0.75 * np.log(max(p, 1e-30))
        assert abs(got[j] - want) <= 2.0 ** -22 * abs(want), (p, got[j], want)
