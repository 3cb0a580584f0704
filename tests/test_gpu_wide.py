"""The fused fan-in-64 sweep.  One pass (batches of up to 16): against the oracle
at widths up to its widest, ragged batches, both losses, positives at and past
the 1024 it keeps on chip, and 16-bit against 32-bit indices bit for bit.
Several passes, which it takes only in layers of 2^29 inputs and more: the
step's first moment, loss and dX against the separate gradient calls (the staged
sweep) of the same layer, in bf16's tolerance, and both index types bit for
bit; the fan-in-32 sweep's passes likewise with the squared hinge and 16-bit
indices."""
import numpy as np
import pytest

import oracle
from paper_2411_03171_amd import ffsl, synth
from tests.parity import RTOL_BF16, assert_close, batch_to_gpu, from_torch_bits, note, to_torch_values, values_f64
from tests.test_gpu_layer import torch_cuda  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

BASE = synth.dataclasses.replace(synth.WORKLOADS["c3_inter2048_L1M"], name="wide", din=0)


def layer_of(torch, W, I, bias, idx16, B, nnz, d, unfused):
    Ix = I.to(torch.int16) if idx16 else I.to(torch.int32)   # columns below 2^15
    return ffsl.SparseLayer(W.clone(), Ix, bias=bias.clone(), B_max=B, nnz_max=max(nnz, 1), unfused=unfused).bind(d)


def snapshot(layer, loss, dX):
    return [from_torch_bits(layer.W, "bf16").copy()] + [t.cpu().numpy().view(np.uint32).copy() for t in
                                                        (layer.m, layer.v, layer.bias, layer.bias_m, loss, dX)]


# (L, d, B, positives, squared hinge, far): far puts most labels past the margin
ONE = [(777, 1024, 1, 3, False, False), (1003, 2048, 11, 60, False, False), (1003, 2048, 16, 1024, False, False),
       (1003, 2048, 16, 1025, False, False), (777, 1024, 16, 80, True, False), (1003, 2048, 11, 50, True, True),
       (515, 128, 16, 1300, True, False), (16, 1920, 5, 0, False, False)]


@pytest.mark.parametrize("case", ONE, ids=["-".join(map(str, c)) for c in ONE])
def test_one_pass(torch_cuda, case):
    torch = torch_cuda
    L, d, B, nnz, hinge, far = case
    w = synth.dataclasses.replace(BASE, L=L, d=d, B=B)
    inp = synth.make_layer_inputs(w, 21)
    rng = np.random.default_rng(21)
    samples = np.sort(rng.integers(0, B, size=nnz))
    off = np.searchsorted(samples, np.arange(B + 1)).astype(np.int64)
    lab = rng.integers(0, L, size=nnz).astype(np.int32)
    bias = (rng.standard_normal(L) * 0.1 - (4.0 if far else 0.0)).astype(np.float32)
    s, b1 = 1.0 / B, 0.9
    off_in, lab_in = off, lab
    if nnz >= 50:   # labels outside [0, L) are ignored
        lab[-2:] = (-1, L)
        off_in, lab_in = np.minimum(off, nnz - 2), lab[:-2]
    ref = oracle.loss_and_grads(values_f64(inp.X, "bf16"), values_f64(inp.W, "bf16"), inp.I, bias.astype(np.float64), off_in, lab_in, s,
                                **({"loss": "sqhinge"} if hinge else {}))
    if far:
        assert (np.abs(ref["g"]).max(axis=0) == 0).mean() > 0.5
    W, I = to_torch_values(inp.W, "bf16", "cuda:0"), torch.from_numpy(inp.I).cuda()
    X, offt, labt = batch_to_gpu(inp.X, off, lab, "bf16")
    runs = []
    for idx16 in (False, True):
        note("wide one pass %s idx16=%s" % (case, idx16))
        layer = layer_of(torch, W, I, torch.from_numpy(bias).cuda(), idx16, B, nnz, d, False)
        loss, dX = layer.train_step(X, offt, labt, t=1, s=s, beta1=b1, lr=1e-3, flags=ffsl.FFSL_LOSS_SQHINGE if hinge else 0)
        torch.cuda.synchronize()
        runs.append(snapshot(layer, loss, dX))
        if not idx16:
            assert_close(loss.cpu().numpy()[0], ref["loss"], RTOL_BF16, "loss")
            assert_close(dX.cpu().numpy(), ref["dX"], RTOL_BF16, "dX")
            assert_close(layer.m.cpu().numpy() / (1.0 - b1), ref["dW"], RTOL_BF16, "dW")
            assert_close(layer.bias_m.cpu().numpy() / (1.0 - b1), ref["dbias"], RTOL_BF16, "dbias")
            Wref = values_f64(inp.W, "bf16") - 1e-3 * np.sign(layer.m.cpu().numpy())   # a first step is lr sign(g)
            assert_close(values_f64(from_torch_bits(layer.W, "bf16"), "bf16"), Wref, RTOL_BF16, "W")
    for a, b in zip(*runs):
        assert np.array_equal(a, b)


# (L, d, k, B, positives, squared hinge): two and three passes of 16 samples; of
# 64 samples two and three at fan-in 32
MANY = [(524288, 2048, 64, 17, 80, False), (262144, 2048, 64, 40, 200, True), (262150, 2048, 64, 48, 1500, False),
        ((1 << 18) + 9, 128, 32, 140, 600, True), ((1 << 18) + 9, 384, 32, 70, 1300, True)]


@pytest.mark.parametrize("case", MANY, ids=["-".join(map(str, c)) for c in MANY])
def test_several_passes(torch_cuda, case):
    torch = torch_cuda
    L, d, k, B, nnz, hinge = case
    g = torch.Generator(device="cuda:0").manual_seed(5)
    rand = lambda *s: torch.rand(*s, generator=g, device="cuda:0")
    W = ((rand(L, k) * 2 - 1) / k ** 0.5).to(torch.bfloat16)
    I = torch.arange(k, device="cuda:0")[None] * (d // k) + (rand(L, k) * (d // k)).long()
    bias = rand(L) * 0.2 - 0.5
    X = torch.randn(B, d, generator=g, device="cuda:0").to(torch.bfloat16)
    off = torch.linspace(0, nnz, B + 1, device="cuda:0").int()
    lab = (rand(nnz) * L).int()
    flags = ffsl.FFSL_LOSS_SQHINGE if hinge else 0
    note("several passes %s, separate calls" % (case,))
    ref = layer_of(torch, W, I, bias, False, B, nnz, d, True)
    rloss = torch.empty(1, device="cuda:0")
    rdX = ref.backward(X, off, lab, loss_out=rloss, flags=flags)

    def close(got, want, what):
        assert bool(torch.isfinite(got).all()), what
        assert float((got - want).abs().max()) <= RTOL_BF16 * float(want.abs().max()), what
        assert float((got - want).norm()) <= RTOL_BF16 * float(want.norm()), what

    runs = []
    for idx16 in (False, True):
        note("several passes %s idx16=%s" % (case, idx16))
        layer = layer_of(torch, W, I, bias, idx16, B, nnz, d, False)
        loss, dX = layer.train_step(X, off, lab, t=1, beta1=0.9, flags=flags)
        if not idx16:
            close(loss, rloss, "loss")
            close(dX, rdX, "dX")
            close(layer.m / 0.1, ref.dW, "dW")
            close(layer.bias_m / 0.1, ref.dbias, "dbias")
        runs.append([t.clone() for t in (layer.W, layer.m, layer.v, layer.bias, layer.bias_m, loss, dX)])
    for a, b in zip(*runs):
        assert torch.equal(a, b)
