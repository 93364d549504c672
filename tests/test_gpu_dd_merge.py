"""Merges over runs of memory (the merged qubits lowest): shortest and longer
runs of the vector path, one and several chunks per output, FP32 and FP64
entries, entries at a 4- or 8-byte aligned address.  The bins of one recursion
against the oracle's full output summed over the merged qubits, relative L1
1e-6 (FP32 entries and arithmetic) and 1e-12 (FP64)."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import fd, metrics
from tests.gpu_util import oracle_inputs

pytestmark = pytest.mark.gpu
cqc = pytest.importorskip("paper_2012_02333_amd")


@pytest.mark.parametrize("prec,np_dt,bar", [("fp32", np.float32, 1e-6), ("fp64", np.float64, 1e-12)])
@pytest.mark.parametrize("f1,n_active", [(9, 6), (10, 6), (11, 6), (12, 7), (13, 6), (14, 6), (14, 8)])
def test_dd_merge_runs(f1, n_active, prec, np_dt, bar):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n = 6 + f1
    cut = W.CutMap(n, [6, f1], [0], [1], list(range(n)))
    host = [np.abs(E).astype(np_dt) for E in W.random_entries(cut, seed=1000 + f1)]
    dev = []
    for E in host:   # one element past the allocation's alignment
        buf = torch.empty(E.size + 1, dtype=torch.from_numpy(E).dtype, device="cuda")
        buf[1:].copy_(torch.from_numpy(E.reshape(-1)))
        dev.append(buf[1:].view(E.shape))
    bins, recs = cqc.reconstruct_dd(dev, cqc.CutMap.from_workload(cut), n_active, 1, precision=prec)
    ref = fd.reconstruct(oracle_inputs(host), cut).reshape(2 ** n_active, -1).sum(axis=1)
    assert metrics.rel_l1(bins[0].cpu().numpy(), ref) <= bar
    assert abs(recs[0]["mass"] - ref.sum()) <= bar * ref.sum()
