"""The staged sweep (scores, dX and dW as three kernels) at the sizes where its
tiles and units can go wrong: every batch tile and sub-tile width, fan-ins at
the edges of a unit, ragged rows and samples, several slabs of rows.

Operands are exact in the matrix products (bf16 weights and inputs, the loss
gradient and fp32 inputs split into bf16 planes that add up to it), so both
value types are held to the fp32 tolerance."""
import numpy as np
import pytest

from paper_2411_03171_amd import synth
from tests.parity import RTOL_BF16, RTOL_F32, assert_close, batch_to_gpu, make_gpu_layer, note, values_f64
from tests.test_gpu_layer import oracle_grads, torch_cuda  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

BASE = synth.WORKLOADS["c4_bf16_L3M"]


def shape(value, L, d, k, B, mean_pos=4.0):
    return synth.dataclasses.replace(BASE, name="staged", value=value, L=L, d=d, k=k, B=B, mean_pos=mean_pos)


# (value, L, d, k, B)
CASES = [
    # bf16: tiles of 64, 32 and 16 samples by batch and by width; fan-ins
    # around a unit's 16, 32, 64 and a row's 128 slots; widths off 16 and 128
    ("bf16", 1, 768, 32, 33), ("bf16", 67, 129, 1, 64), ("bf16", 333, 257, 15, 65), ("bf16", 130, 768, 17, 31),
    ("bf16", 259, 769, 33, 70), ("bf16", 514, 1151, 64, 16), ("bf16", 131, 1152, 65, 40), ("bf16", 95, 2303, 100, 47),
    ("bf16", 66, 2304, 127, 18), ("bf16", 200, 4607, 128, 5), ("bf16", 1030, 640, 128, 130),
    # fp32: tiles of 32 and 16, split into 32, 16 and 8 for dW
    ("f32", 3, 130, 2, 1), ("f32", 515, 768, 16, 33), ("f32", 190, 832, 31, 64), ("f32", 77, 833, 32, 47),
    ("f32", 301, 1151, 64, 20), ("f32", 65, 1152, 96, 17), ("f32", 129, 1249, 128, 50), ("f32", 40, 2303, 3, 24),
]


def inputs(w, seed):
    inp = synth.make_layer_inputs(w, seed)
    bias = (np.random.default_rng(seed).standard_normal(w.L) * 0.3 - 1.0).astype(np.float32)
    return inp, bias


def grads(torch, w, inp, bias, flags=0):
    layer = make_gpu_layer(inp, w, bias_values=bias)
    X, off, lab = batch_to_gpu(inp.X, inp.off, inp.lab, w.value)
    loss = torch.empty(1, device="cuda:0")
    dX = layer.backward(X, off, lab, loss_out=loss, flags=flags)
    fwd, z = layer.forward_loss(X, off, lab, logits=True, flags=flags)
    torch.cuda.synchronize()
    return layer, loss, dX, fwd, z


@pytest.mark.parametrize("case", CASES, ids=["-".join(map(str, c)) for c in CASES])
def test_gradients_at_the_edges(torch_cuda, case):
    w = shape(*case)
    note("staged %s" % (case,))
    inp, bias = inputs(w, 3)
    layer, loss, dX, fwd, z = grads(torch_cuda, w, inp, bias)
    ref = oracle_grads(w, inp, bias, 1.0 / w.B)
    assert_close(z.cpu().numpy(), ref["z"], RTOL_F32, "logits")
    assert_close(fwd.cpu().numpy()[0], ref["loss"], RTOL_F32, "loss")
    assert_close(loss.cpu().numpy()[0], ref["loss"], RTOL_F32, "loss of the backward call")
    assert_close(layer.dW.cpu().numpy(), ref["dW"], RTOL_F32, "dW")
    assert_close(layer.dbias.cpu().numpy(), ref["dbias"], RTOL_F32, "dbias")
    assert_close(dX.cpu().numpy(), ref["dX"], RTOL_F32, "dX")


@pytest.mark.parametrize("value", ["bf16", "f32"])
def test_several_slabs_and_many_positives(torch_cuda, value):
    """1024 samples' gradients fill a slab with about 20 thousand rows; 30
    positives a sample are more than a workgroup lists at once."""
    w = shape(value, 43011, 40, 3, 1024, mean_pos=30.0)
    note("staged slabs %s" % value)
    inp, bias = inputs(w, 4)
    layer, loss, dX, fwd, _ = grads(torch_cuda, w, inp, bias)
    ref = oracle_grads(w, inp, bias, 1.0 / w.B)
    assert_close(fwd.cpu().numpy()[0], ref["loss"], RTOL_F32, "loss")
    assert_close(loss.cpu().numpy()[0], ref["loss"], RTOL_F32, "loss of the backward call")
    assert_close(layer.dW.cpu().numpy(), ref["dW"], RTOL_F32, "dW")
    assert_close(layer.dbias.cpu().numpy(), ref["dbias"], RTOL_F32, "dbias")
    assert_close(dX.cpu().numpy(), ref["dX"], RTOL_F32, "dX")


@pytest.mark.parametrize("value,k", [("bf16", 12), ("bf16", 100), ("f32", 12), ("f32", 40)])
def test_repeated_columns_count_twice(torch_cuda, value, k):
    """A column that a row holds more than once contributes every time.  In a
    bf16 layer the dX product takes the sum of its weights rounded to bf16."""
    w = shape(value, 517, 300, k, 40)
    inp, bias = inputs(w, 5)
    I = inp.I.copy()
    I[::3, 1] = I[::3, 0]
    I[::3, k - 1] = I[::3, 0]
    I[1::3, 9] = I[1::3, 8]
    inp = synth.dataclasses.replace(inp, I=I)
    note("staged repeated columns %s k=%d" % (value, k))
    layer, loss, dX, fwd, z = grads(torch_cuda, w, inp, bias)
    ref = oracle_grads(w, inp, bias, 1.0 / w.B)
    assert_close(z.cpu().numpy(), ref["z"], RTOL_F32, "logits")
    assert_close(layer.dW.cpu().numpy(), ref["dW"], RTOL_F32, "dW")
    assert_close(dX.cpu().numpy(), ref["dX"], RTOL_BF16 if value == "bf16" else RTOL_F32, "dX")


@pytest.mark.parametrize("value", ["bf16", "f32"])
def test_a_non_finite_weight_stays_in_its_row(torch_cuda, value):
    """A NaN weight makes its row's scores and gradients NaN; of dX only the
    columns the row holds, in every sample."""
    torch = torch_cuda
    w = shape(value, 200, 160, 16, 70)
    inp, bias = inputs(w, 6)
    Wb = inp.W.copy()
    Wb[77, 3] = np.nan if value == "f32" else 0x7FC0
    inp = synth.dataclasses.replace(inp, W=Wb)
    note("staged NaN weight %s" % value)
    layer, loss, dX, fwd, z = grads(torch, w, inp, bias)
    held = np.zeros(w.d, bool)
    held[inp.I[77]] = True
    assert np.isnan(fwd.cpu().numpy()[0]) and np.isnan(loss.cpu().numpy()[0])
    dXg, dWg = dX.cpu().numpy(), layer.dW.cpu().numpy()
    assert np.isnan(dXg[:, held]).all() and np.isfinite(dXg[:, ~held]).all()
    assert np.isnan(dWg[77]).all() and np.isfinite(np.delete(dWg, 77, axis=0)).all()


@pytest.mark.parametrize("value", ["bf16", "f32"])
@pytest.mark.parametrize("L,k", [(253, 16), (254, 11), (255, 3), (251, 17), (253, 32)])
def test_rows_past_the_end_are_left_alone(torch_cuda, value, L, k):
    """The layer's arrays are the leading L rows of larger ones: what lies past
    them keeps its bits, in the stored-gradient and in the Adam mode (the last
    unit of dW holds fewer rows than the others)."""
    torch = torch_cuda
    w = shape(value, L, 96, k, 33)
    inp, bias = inputs(w, 8)
    note("staged tail L=%d k=%d %s" % (L, k, value))
    layer = make_gpu_layer(inp, w, bias_values=bias)
    layer.close()
    names = ["W", "I", "m", "v", "dW", "bias", "bias_m", "bias_v", "dbias"]
    big = {}
    for n in names:
        t = getattr(layer, n)
        big[n] = torch.full((L + 5,) + tuple(t.shape[1:]), 7, dtype=t.dtype, device=t.device)
        big[n][:L] = t
        setattr(layer, n, big[n][:L])
    layer.bind(w.d)
    X, off, lab = batch_to_gpu(inp.X, inp.off, inp.lab, w.value)
    layer.dW.fill_(np.nan)
    layer.backward(X, off, lab)
    layer.train_step(X, off, lab, t=2)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(layer.dW).all())
    for n in names:
        assert bool((big[n][L:] == 7).all()), n
