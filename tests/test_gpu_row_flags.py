"""Row flags (early termination) over every layout of the flag pass: rows of one
column to several chunks, row counts that leave the last wave partly filled,
FP32 and FP64.  A term whose row is flagged dead is skipped, so a live row
flagged dead, or its neighbour's flag taken for it, changes the outputs: each
row has one non-zero element, at another place in each, or none."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import fd
from tests.gpu_util import oracle_inputs, abs_bound, elementwise_ok, U32, U64

pytestmark = pytest.mark.gpu
cqc = pytest.importorskip("paper_2012_02333_amd")


@pytest.mark.parametrize("prec,np_dt,unit", [("fp32", np.float32, U32), ("fp64", np.float64, U64)])
@pytest.mark.parametrize("f", [(0, 9), (1, 8), (2, 7), (3, 9), (6, 6), (8, 5), (9, 4), (10, 3), (11, 2), (12, 1), (13, 0)])
def test_row_flags_layouts(f, prec, np_dt, unit):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    cut = W.CutMap(sum(f), list(f), [0, 0, 0], [1, 1, 1], list(range(sum(f))))
    rng = np.random.default_rng(1100 + f[0])
    host = []
    for c in range(2):
        rows, w = cut.entry_shape(c)
        E = np.zeros((rows, w), dtype=np_dt)
        for r in range(rows):
            if r % 5 != 2:
                E[r, rng.integers(0, w) if r % 3 else w - 1] = rng.uniform(0.5, 1.0)
        host.append(E)
    dev = [torch.from_numpy(E).cuda() for E in host]
    p, _ = cqc.reconstruct_fd(dev, cqc.CutMap.from_workload(cut), precision=prec)
    e64 = oracle_inputs(host)
    ok, info = elementwise_ok(p.double().cpu().numpy(), fd.reconstruct(e64, cut), abs_bound(e64, cut), unit, 64)
    assert ok, info
