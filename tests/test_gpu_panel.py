"""GPU parity of the panel contraction kernels (FP32 steps of three shared cuts
in registers, of four and more streamed; at least 2^22 outputs in a single call and 2^19 in a batch): panels and row
runs at their smallest, live-term counts at and around the kernel's groups of
eight, row flags read by the waves or through the label lists, batched
intermediate steps, and the batched cross-entropy form.  Elementwise bound as in test_gpu_fd; sums in FP64 (n outputs of relative rounding 2^-53
each leave at most n 2^-53 of the sum of magnitudes, 1e-12 here)."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import fd
from tests.gpu_util import to_dev, oracle_inputs, abs_bound, elementwise_ok, U32

pytestmark = pytest.mark.gpu
cqc = pytest.importorskip("paper_2012_02333_amd")


def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _entries(cut, seed, live):
    """Random entries of which sub 0 keeps `live` rows (spread over all of them)."""
    rows = cut.entry_shape(0)[0]
    keep = set(np.linspace(0, rows - 1, live).astype(int)) if live else set()
    return W.random_entries(cut, seed=seed, zero_rows=[(0, r) for r in range(rows) if r not in keep])


def _check(cut, p, host, seed):
    xs = W.sample_outputs(cut.n, 2048, seed=seed)
    e64 = oracle_inputs(host)
    got = p[torch.from_numpy(xs).to("cuda")].double().cpu().numpy()
    ok, info = elementwise_ok(got, fd.reconstruct(e64, cut, xs), abs_bound(e64, cut, xs), U32, 4 ** cut.n_cuts)
    assert ok, info


@pytest.mark.parametrize("f,live", [((11, 11), 64), ((11, 11), 63), ((11, 11), 9), ((11, 11), 8), ((11, 11), 1),
                                    ((11, 11), 0), ((6, 16), 64), ((6, 16), 37), ((16, 6), 64), ((16, 6), 21),
                                    ((15, 8), 40)])
def test_panel_step(f, live):
    _gpu()
    n = sum(f)
    cut = W.CutMap(n, list(f), [0, 0, 0], [1, 1, 1], list(range(n)))
    host, dev = to_dev(_entries(cut, 900 + live, live), torch.float32)
    with cqc.trace() as tr:
        p, mass = cqc.reconstruct_fd(dev, cqc.CutMap.from_workload(cut), precision="fp32")
        torch.cuda.synchronize()
    assert "wide_f32_final_panel" in tr.result, tr.result
    _check(cut, p, host, 901)
    s, sa = float(p.double().sum()), float(p.double().abs().sum())
    assert abs(float(mass) - s) <= 1e-12 * sa
    if live == 0:
        assert sa == 0.0


@pytest.mark.parametrize("f,k,live", [((11, 11), 4, 256), ((11, 11), 4, 33), ((11, 11), 4, 32), ((11, 11), 4, 31),
                                      ((11, 11), 4, 1), ((11, 11), 4, 0), ((6, 16), 4, 100), ((16, 6), 4, 64),
                                      ((15, 7), 4, 200), ((11, 11), 5, 1000)])
def test_stream_step(f, k, live):
    """Four and five shared cuts: the streamed form, with one panel or one row tile at its narrowest."""
    _gpu()
    n = sum(f)
    cut = W.CutMap(n, list(f), [0] * k, [1] * k, list(range(n)))
    host, dev = to_dev(_entries(cut, 940 + live, live), torch.float32)
    with cqc.trace() as tr:
        p, mass = cqc.reconstruct_fd(dev, cqc.CutMap.from_workload(cut), precision="fp32")
        torch.cuda.synchronize()
    assert "wide_f32_final_stream" in tr.result, tr.result
    _check(cut, p, host, 941)
    s, sa = float(p.double().sum()), float(p.double().abs().sum())
    assert abs(float(mass) - s) <= 1e-12 * sa
    if live == 0:
        assert sa == 0.0


def test_panel_intermediate_and_final():
    """A chain whose intermediate (64 batch entries, some without a live term) and final steps are panels."""
    _gpu()
    cut = W.CutMap(24, [8, 8, 8], [0, 0, 0, 1, 1, 1], [1, 1, 1, 2, 2, 2], list(range(24)))
    ents = W.random_entries(cut, seed=910, zero_rows=[(1, r) for r in range(4096) if r % 64 in (3, 17, 62)])
    host, dev = to_dev(ents, torch.float32)
    with cqc.trace() as tr:
        p, _ = cqc.reconstruct_fd(dev, cqc.CutMap.from_workload(cut), precision="fp32")
        torch.cuda.synchronize()
    assert "wide_f32_inter_panel" in tr.result and "wide_f32_final_panel" in tr.result, tr.result
    _check(cut, p, host, 911)


@pytest.mark.parametrize("keep", [True, False])
@pytest.mark.parametrize("loss", [True, False])
def test_panel_batch_xent(keep, loss):
    """The cross-entropy form writes the two-pass gradient bit for bit; the
    loss terms carry an FP32 logarithm (at most 2 ulp: 2^-22 of each term)."""
    _gpu()
    shapes = [((10, 10), 3, 64), ((6, 13), 3, 40), ((9, 10), 3, 9), ((13, 7), 3, 0),
              ((10, 10), 4, 256), ((6, 13), 4, 65), ((13, 6), 4, 0)]
    cuts_w = [W.CutMap(sum(f), list(f), [0] * k, [1] * k, list(range(sum(f)))) for f, k, _ in shapes]
    dev = [to_dev([np.abs(E) for E in _entries(c, 920 + i, live)], torch.float32)[1]
           for i, (c, (_, _, live)) in enumerate(zip(cuts_w, shapes))]
    cuts = [cqc.CutMap.from_workload(c) for c in cuts_w]
    t = [torch.from_numpy(W.dirichlet_target(c.n, 930 + i).astype(np.float32)).cuda() for i, c in enumerate(cuts_w)]
    plain = cqc.Batch(dev, cuts, precision="fp32")
    plain.run()
    batch = cqc.Batch(dev, cuts, precision="fp32", targets=t, with_loss=loss, keep_outputs=keep)
    for _ in range(2):
        batch.run()
    torch.cuda.synchronize()
    for i in range(len(cuts)):
        p = plain.outs[i]
        assert torch.equal(batch.grads[i], cqc.xent_grad(p, t[i])), i
        if keep:
            assert torch.equal(batch.outs[i], p), i
        if loss:
            term = t[i].double() * p.double().clamp_min(1e-30).log()
            assert abs(float(batch.losses[i]) + float(term.sum())) <= 2.0 ** -22 * float(term.abs().sum()), i
        else:
            assert abs(float(batch.mass[i]) - float(p.double().sum())) <= 1e-12 * float(p.double().abs().sum()), i


@pytest.mark.parametrize("f,k", [((10, 10), 1), ((10, 10), 2), ((10, 12), 3), ((10, 12), 4)])
def test_outputs_and_targets_at_4_byte_alignment(f, k):
    """Row, panel and stream kernels with every caller buffer one element past
    its alignment: the outputs and gradients of aligned buffers, bit for bit,
    and nothing written before or after."""
    _gpu()
    n = sum(f)
    cut_w = W.CutMap(n, list(f), [0] * k, [1] * k, list(range(n)))
    cut = cqc.CutMap.from_workload(cut_w)
    dev = to_dev([np.abs(E) for E in W.random_entries(cut_w, seed=1200 + k)], torch.float32)[1]

    def shifted(x):
        buf = torch.full((x.numel() + 2,), 7.0, device="cuda")
        buf[1:-1].copy_(x.reshape(-1))
        return buf, buf[1:-1].view(x.shape)

    t = torch.from_numpy(W.dirichlet_target(n, 1210).astype(np.float32)).cuda()
    ents = [shifted(E)[1] for E in dev]
    bo, out = shifted(torch.zeros(2 ** n, device="cuda"))
    bg, grad = shifted(torch.zeros(2 ** n, device="cuda"))
    call = cqc.FDCall(ents, cut, "fp32", outs=[out])
    call.run()
    p, mass = cqc.reconstruct_fd(dev, cut, precision="fp32")
    assert torch.equal(out, p) and float(call.mass[0]) == float(mass)
    batch = cqc.Batch([ents, ents], [cut, cut], precision="fp32", targets=[shifted(t)[1], t],
                      grads=[grad, torch.empty_like(t)], keep_outputs=False)
    batch.run()
    assert torch.equal(batch.grads[0], cqc.xent_grad(p, t)) and torch.equal(batch.grads[0], batch.grads[1])
    for b in (bo, bg):
        assert float(b[0]) == 7.0 and float(b[-1]) == 7.0


@pytest.mark.parametrize("f,count", [((10, 10), 2), ((11, 11), 2), ((11, 12), 2), ((12, 12), 2), ((13, 12), 1)])
def test_panel_batch_runs(f, count):
    """Batches whose units take one, two, four and eight row tiles (the launch's
    tile count decides), next to an instance with a single row tile: the single
    call's outputs bit for bit where that runs panels too, and the oracle's."""
    _gpu()
    shapes = [f] * count + [(6, 13)]
    cuts_w = [W.CutMap(sum(s), list(s), [0] * 3, [1] * 3, list(range(sum(s)))) for s in shapes]
    hosts, dev = zip(*[to_dev(_entries(c, 990 + i, 60), torch.float32) for i, c in enumerate(cuts_w)])
    cuts = [cqc.CutMap.from_workload(c) for c in cuts_w]
    batch = cqc.Batch(list(dev), cuts, precision="fp32")
    batch.run()
    for i, c in enumerate(cuts):
        _check(cuts_w[i], batch.outs[i], hosts[i], 995 + i)
        s, sa = float(batch.outs[i].double().sum()), float(batch.outs[i].double().abs().sum())
        assert abs(float(batch.mass[i]) - s) <= 1e-12 * sa, i
        if c.n >= 22:
            assert torch.equal(batch.outs[i], cqc.reconstruct_fd(dev[i], c, precision="fp32")[0]), i
