"""The trace tells the batched kernels of a step apart: panel, stream and row
kernels, plain and in the cross-entropy form, and the register kernels."""
import numpy as np
import pytest
import torch

import workloads as W
from tests.gpu_util import to_dev

pytestmark = pytest.mark.gpu
cqc = pytest.importorskip("paper_2012_02333_amd")


@pytest.mark.parametrize("f,k,plain,xent", [
    ((10, 10), 3, "wide_f32_queue", "wide_f32_queue_xent_panel"),
    ((10, 10), 4, "wide_f32_queue_stream", "wide_f32_queue_xent_stream"),
    ((7, 8), 1, "contract_strip_queue", "contract_rows_256_xent"),
    ((8, 7), 1, "contract_rows_128", "contract_rows_128_xent"),
    ((9, 6), 2, "contract_rows_64", "contract_rows_64_xent"),
    ((4, 5), 1, "contract_small_queue", "contract_small_queue_xent")])
def test_batched_kernels_by_name(f, k, plain, xent):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    cut_w = W.CutMap(sum(f), list(f), [0] * k, [1] * k, list(range(sum(f))))
    cut = cqc.CutMap.from_workload(cut_w)
    dev = to_dev([np.abs(E) for E in W.random_entries(cut_w, seed=1500 + k)], torch.float32)[1]
    t = torch.from_numpy(W.dirichlet_target(cut.n, 1501).astype(np.float32)).cuda()
    known = {plain, xent, xent + "_loss"}
    for kw, name in [({}, plain), (dict(targets=[t, t]), xent), (dict(targets=[t, t], with_loss=True), xent)]:
        batch = cqc.Batch([dev, dev], [cut, cut], precision="fp32", **kw)
        with cqc.trace() as tr:
            batch.run()
            torch.cuda.synchronize()
        got = known & set(tr.result)
        assert len(got) == 1 and got.pop().startswith(name), (name, tr.result)
