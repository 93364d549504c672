"""GPU parity of the FP64 row kernel (steps of at most two shared cuts from 2^20
outputs on), seen to run by its trace name: one, four and 16 terms, row tiles
and panels at their smallest, ordinary and non-temporal stores, dead rows, the
batched intermediate step; and of the FP32 form over its run lengths and both
kinds of stores.  Elementwise bound as in test_gpu_fd; sums in FP64 (1e-12 of
the sum of magnitudes)."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import fd
from tests.gpu_util import to_dev, oracle_inputs, abs_bound, elementwise_ok, U32, U64

pytestmark = pytest.mark.gpu
cqc = pytest.importorskip("paper_2012_02333_amd")


def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _run(cut, ents, precision, seed, unit, out=None):
    """One call against the oracle on a sample; -> (p, device entries, cut, trace)."""
    dt = torch.float64 if precision == "fp64" else torch.float32
    host, dev = to_dev(ents, dt)
    c = cqc.CutMap.from_workload(cut)
    with cqc.trace() as tr:
        p, mass = cqc.reconstruct_fd(dev, c, precision=precision, out_dtype=out)
        torch.cuda.synchronize()
    xs = W.sample_outputs(cut.n, 4096, seed=seed)
    e64 = oracle_inputs(host)
    got = p[torch.from_numpy(xs).cuda()].double().cpu().numpy()
    ok, info = elementwise_ok(got, fd.reconstruct(e64, cut, xs), abs_bound(e64, cut, xs), unit, 4 ** cut.n_cuts)
    assert ok, info
    assert abs(float(mass) - float(p.double().sum())) <= 1e-12 * float(p.double().abs().sum())
    return p, dev, c, tr.result


def _pair(f, k):
    return W.CutMap(sum(f), list(f), [0] * k, [1] * k, list(range(sum(f))))


@pytest.mark.parametrize("k", [0, 1, 2])
@pytest.mark.parametrize("f", [(10, 10), (7, 14), (13, 7), (5, 16), (11, 12), (4, 18)])
def test_f64_step(f, k):
    """Its outputs are those of the batched register kernel bit for bit."""
    _gpu()
    cut = _pair(f, k)
    p, dev, c, kt = _run(cut, W.random_entries(cut, seed=1400 + k), "fp64", 1401, U64)
    assert ("contract_rows_f64" in kt) == (f != (4, 18)), kt
    batch = cqc.Batch([dev, dev], [c, c], precision="fp64")
    batch.run()
    assert torch.equal(batch.outs[0], p)


def test_f64_wide_rows_of_16_terms_on_the_register_kernel():
    _gpu()
    cut = _pair((6, 18), 2)
    kt = _run(cut, W.random_entries(cut, seed=1405), "fp64", 1406, U64)[3]
    assert "contract_rows_f64" not in kt and "contract_small_64x256" in kt, kt


@pytest.mark.parametrize("k0,k1", [(1, 3), (2, 3), (3, 1), (2, 2), (1, 1)])
def test_f64_chain(k0, k1):
    """Small-term steps as the batched intermediate and as the final one, with
    dead rows where the plan computes row flags (a step of three cuts)."""
    _gpu()
    f = [8, 9, 8] if k0 < 3 else [8, 8, 9]
    cut = W.CutMap(25, f, [0] * k0 + [1] * k1, [1] * k0 + [2] * k1, list(range(25)))
    zr = [(0, 1), (2, 0), (2, 3)] + [(1, r) for r in range(4 ** (k0 + k1)) if r % 7 == 2]
    p, dev, c, kt = _run(cut, W.random_entries(cut, seed=1410, zero_rows=zr), "fp64", 1411, U64)
    assert any(n.startswith("contract_rows_f64") for n in kt), kt
    batch = cqc.Batch([dev, dev], [c, c], precision="fp64")
    batch.run()
    assert torch.equal(batch.outs[0], p)


@pytest.mark.parametrize("f,k,out", [((12, 14), 0, torch.float32), ((13, 13), 1, torch.float32),
                                     ((14, 12), 0, torch.float32), ((11, 13), 2, torch.float32),
                                     ((12, 13), 2, torch.float32), ((7, 18), 2, torch.float32),
                                     ((12, 12), 1, torch.float32), ((11, 12), 2, torch.float64),
                                     ((16, 7), 0, torch.float64), ((13, 14), 1, torch.float32)])
def test_f32_run_lengths_and_stores(f, k, out):
    _gpu()
    cut = _pair(f, k)
    kt = _run(cut, W.random_entries(cut, seed=1420 + k), "fp32", 1421, U32, out)[3]
    assert any(n.startswith(("contract_small_rows", "contract_small_strip")) for n in kt), kt
