"""Batched steps that run the same kernel share one launch, whatever tile shape
the planner gave them."""
import pytest
import torch

import workloads as W
from tests.gpu_util import to_dev

pytestmark = pytest.mark.gpu
cqc = pytest.importorskip("paper_2012_02333_amd")


@pytest.mark.parametrize("shapes,name", [([(4, 10), (5, 9), (7, 10)], "contract_strip_queue"),
                                         ([(4, 10), (5, 9), (7, 10), (3, 5)], "contract_strip_queue")])
def test_row_steps_of_every_tile_in_one_launch(shapes, name):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    cuts_w = [W.CutMap(sum(f), list(f), [0], [1], list(range(sum(f)))) for f in shapes]
    ents = [to_dev(W.random_entries(c, seed=1300 + i), torch.float32)[1] for i, c in enumerate(cuts_w)]
    cuts = [cqc.CutMap.from_workload(c) for c in cuts_w]
    batch = cqc.Batch(ents, cuts, precision="fp32")
    with cqc.trace() as tr:
        batch.run()
        torch.cuda.synchronize()
    assert tr.result[name][0] == 1, tr.result
    for i, c in enumerate(cuts):
        p, mass = cqc.reconstruct_fd(ents[i], c, precision="fp32")
        assert torch.equal(batch.outs[i], p), i
        assert abs(float(batch.mass[i]) - float(mass)) <= 1e-12 * max(1.0, float(p.double().abs().sum())), i
