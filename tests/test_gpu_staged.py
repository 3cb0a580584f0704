"""The staged sweep (scores, dX and dW as three kernels) at the sizes where its
tiles and units can go wrong: every batch tile and sub-tile width, fan-ins at
the edges of a unit, ragged rows and samples, several slabs of rows.

Operands are exact in the matrix products (bf16 weights and inputs, the loss
gradient and fp32 inputs split into bf16 planes that add up to it), so both
value types are held to the fp32 tolerance."""
import numpy as np
import pytest

from paper_2411_03171_amd import synth
from tests.parity import RTOL_F32, assert_close, batch_to_gpu, from_torch_bits, make_gpu_layer, note, values_f64
from tests.test_gpu_layer import adam_reference, oracle_grads, torch_cuda  # noqa: F401  (fixture)

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
    """A column that a row holds more than once contributes every time, whichever
    of its weights are zero."""
    w = shape(value, 517, 300, k, 40)
    inp, bias = inputs(w, 5)
    I, Wb = inp.I.copy(), inp.W.copy()
    I[::3, 1] = I[::3, 0]
    I[::3, k - 1] = I[::3, 0]
    I[1::3, 9] = I[1::3, 8]
    Wb[::6, 0], Wb[::9, 1], Wb[::12, k - 1], Wb[1::6, 8], Wb[4::6, 9] = 0, 0, 0, 0, 0
    inp = synth.dataclasses.replace(inp, I=I, W=Wb)
    note("staged repeated columns %s k=%d" % (value, k))
    layer, loss, dX, fwd, z = grads(torch_cuda, w, inp, bias)
    ref = oracle_grads(w, inp, bias, 1.0 / w.B)
    assert_close(z.cpu().numpy(), ref["z"], RTOL_F32, "logits")
    assert_close(layer.dW.cpu().numpy(), ref["dW"], RTOL_F32, "dW")
    assert_close(dX.cpu().numpy(), ref["dX"], RTOL_F32, "dX")
    again = grads(torch_cuda, w, inp, bias)[2]
    assert np.array_equal(dX.cpu().numpy().view(np.uint32), again.cpu().numpy().view(np.uint32))


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


# (value, L, d, k, B): every scoring tile, one and three planes of g, positives
# of more rows than a segment of targets holds (the last two)
SETTLED = [("bf16", 300, 64, 12, 33), ("bf16", 300, 768, 32, 70), ("bf16", 290, 96, 40, 9), ("bf16", 300, 400, 8, 24),
           ("f32", 300, 64, 12, 33), ("f32", 311, 700, 40, 9), ("bf16", 600011, 1151, 2, 64), ("f32", 1300003, 2303, 2, 12)]


def settled(case, hinge):
    """Every pair far on its right side: column 0, held by every row, is +-c in
    a sample and the row's weight there +-1; a row's positives are the samples
    of its sign, all others negatives.  One pair in three is no target, so some
    rows stay unsettled."""
    value, L, d, k, B = case
    w = shape(value, L, d, k, B)
    rng = np.random.default_rng(12)
    I = np.stack([np.zeros(L, np.int64)] + [1 + (rng.integers(0, d - 1, L) + j * ((d - 1) // k)) % (d - 1)
                                            for j in range(k - 1)], axis=1).astype(np.int32)
    Wv = rng.standard_normal((L, k)).astype(np.float32) * 1e-3
    Wv[:, 0] = np.where(np.arange(L) % 2 == 0, 1.0, -1.0)
    X = rng.standard_normal((B, d)).astype(np.float32)
    c = 2.0 if hinge else 24.0
    X[:, 0] = np.where(np.arange(B) % 3 == 0, c, -c)
    bias = (rng.standard_normal(L) * 0.01).astype(np.float32)
    rows = np.arange(L) if L < 1000 else np.concatenate([np.arange(200), rng.integers(0, L, 100), [L - 1]])
    per = [np.unique(rows[Wv[rows, 0] * X[b, 0] > 0]) for b in range(B)]
    if L >= 1000:   # elsewhere a row has no positive: give it negative scores only
        quiet = np.ones(L, bool)
        quiet[rows] = False
        Wv[quiet, 0] = 0.0
        bias[quiet] -= c
    off = np.concatenate([[0], np.cumsum([len(p) for p in per])]).astype(np.int64)
    lab = np.concatenate(per).astype(np.int32)
    bits = (lambda a: synth.f32_to_bf16_bits(a)) if value == "bf16" else (lambda a: a)
    inp = synth.dataclasses.replace(synth.make_layer_inputs(shape(value, 8, d, k, B), 1), X=bits(X), W=bits(Wv), I=I, off=off, lab=lab,
                                    bias=bias)
    return w, inp, bias


@pytest.mark.parametrize("case", SETTLED, ids=["-".join(map(str, c)) for c in SETTLED])
def test_settled_positives_leave_nothing(torch_cuda, case):
    """Squared hinge past the margin everywhere: the loss and every gradient are
    exactly zero, and a step leaves weights and biases as they are."""
    torch = torch_cuda
    from paper_2411_03171_amd import ffsl
    w, inp, bias = settled(case, True)
    note("staged settled hinge %s" % (case,))
    layer, loss, dX, fwd, z = grads(torch, w, inp, bias, flags=ffsl.FFSL_LOSS_SQHINGE)
    for t in (loss, fwd, layer.dW, layer.dbias, dX):
        assert bool((t == 0).all())
    X, off, lab = batch_to_gpu(inp.X, inp.off, inp.lab, w.value)
    W0, b0 = layer.W.clone(), layer.bias.clone()
    loss, dX = layer.train_step(X, off, lab, t=1, lr=1e-2, flags=ffsl.FFSL_LOSS_SQHINGE)
    assert bool((loss == 0).all()) and bool((dX == 0).all())
    assert torch.equal(layer.W, W0) and torch.equal(layer.bias, b0)


@pytest.mark.parametrize("case", SETTLED, ids=["-".join(map(str, c)) for c in SETTLED])
def test_loss_of_settled_positives(torch_cuda, case):
    """BCE of pairs with |z| about 24 on the right side, some ten orders below the
    scores: held to the relative error of exp at that z, a few units of z's last
    place (2^-20 each, z being a sum of k terms)."""
    w, inp, bias = settled(case, False)
    note("staged settled BCE %s" % (case,))
    layer, loss, dX, fwd, z = grads(torch_cuda, w, inp, bias)
    if w.L < 1000:
        zz = oracle_grads(w, inp, bias, 1.0 / w.B)["z"]
    else:
        zz = z.cpu().numpy().astype(np.float64)
    y = np.zeros((w.B, w.L), bool)
    for b in range(w.B):
        y[b, inp.lab[inp.off[b]:inp.off[b + 1]]] = True
    e = np.exp(-np.abs(zz))
    assert (np.where(y, zz, -zz) > 20).all()
    want = np.log1p(e).sum() / w.B
    assert abs(fwd.cpu().numpy()[0] - want) <= 1e-5 * want
    assert abs(loss.cpu().numpy()[0] - want) <= 1e-5 * want


def test_positives_of_one_sample_cost_what_those_of_many_do(torch_cuda):
    """100 thousand positives in one sample, against as many over all samples:
    the preparation must not compare a sample's labels with each other (that
    took hundreds of times as long).  And a label given twice counts once."""
    torch = torch_cuda
    L, B, n = 200003, 32, 100000
    w = shape("bf16", L, 64, 4, B)
    rng = np.random.default_rng(3)
    inp, bias = inputs(w, 9)
    lab = rng.permutation(L)[:n].astype(np.int32)
    one = np.full(B + 1, n, np.int64)
    one[0] = 0
    many = np.linspace(0, n, B + 1).astype(np.int64)
    layer = make_gpu_layer(inp, w, bias_values=bias, nnz_max=2 * n)

    def run(off, lab):
        X, offt, labt = batch_to_gpu(inp.X, off, lab, w.value)
        ts = []
        for _ in range(4):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            loss = layer.forward_loss(X, offt, labt)
            e1.record()
            torch.cuda.synchronize()
            ts.append(e0.elapsed_time(e1))
        return min(ts), loss.cpu().numpy()[0]

    note("staged positives of one sample")
    t_many, _ = run(many, lab)
    t_one, loss_one = run(one, lab)
    assert t_one < 5.0 * t_many, (t_one, t_many)
    twice = np.concatenate([lab, lab[::-1]])
    off2 = one * 2
    _, loss_two = run(off2, twice)
    assert loss_one == loss_two


def plain_grads(w, inp, bias, hinge):
    """z, g, dW, dbias and dX term by term in float64, with the infinities and
    NaNs that the terms and sums give."""
    X, W = values_f64(inp.X, w.value), values_f64(inp.W, w.value)
    y = np.zeros((w.B, w.L), bool)
    for b in range(w.B):
        y[b, inp.lab[inp.off[b]:inp.off[b + 1]]] = True
    with np.errstate(all="ignore"):   # (a sum of both infinities is NaN)
        Xg = X[:, inp.I]                                     # [B, L, k]
        z = (Xg * W[None]).sum(2) + bias[None].astype(np.float64)
        if hinge:
            yh = np.where(y, 1.0, -1.0)
            g = -2.0 * yh * np.fmax(1.0 - yh * z, 0.0) / w.B
        else:
            e = np.exp(-np.abs(z))
            g = (np.where(z >= 0, 1.0 / (1.0 + e), e / (1.0 + e)) - y) / w.B
        dW = (g[:, :, None] * Xg).sum(0)
        dX = np.zeros((w.B, w.d))
        for b in range(w.B):
            np.add.at(dX[b], inp.I, g[b][:, None] * W)
        db = g.sum(0)
    return z, g, dW, db, dX


def same_with_infinities(got, ref, rtol, what):
    got, ref = np.asarray(got, np.float64), np.asarray(ref, np.float64)
    assert np.array_equal(np.isnan(got), np.isnan(ref)), what
    inf = np.isinf(ref)
    assert np.array_equal(got[inf], ref[inf]), what
    fin = np.isfinite(ref)
    assert_close(got[fin], ref[fin], rtol, what)


# (value, L, d, k, B, hinge, fused): one and three planes of g, both value types
# with every sub-tile of dW, in the stored-gradient and in the Adam mode (whose
# dX is that of the weights before the update)
INF = [("bf16", 200, 160, 16, 70, False, False), ("f32", 200, 160, 16, 70, False, False),
       ("bf16", 133, 768, 32, 70, True, True), ("bf16", 133, 300, 100, 20, False, True),
       ("bf16", 200, 160, 16, 70, True, False), ("bf16", 131, 2000, 70, 9, True, False),
       ("f32", 200, 160, 24, 33, True, False), ("f32", 200, 1000, 40, 30, True, True),
       ("f32", 90, 2000, 100, 20, True, False), ("f32", 200, 700, 7, 20, True, False)]


@pytest.mark.parametrize("where", ["weight", "input"])
@pytest.mark.parametrize("case", INF, ids=["-".join(map(str, c)) for c in INF])
def test_infinities(torch_cuda, case, where):
    """An infinite weight makes its row's scores infinite of either sign, an
    infinite input those of the rows that hold its column; with the squared hinge
    so are their g.  Sums that hold such a term are infinite or NaN as the term
    and the sum are, and nothing else is."""
    value, L, d, k, B, hinge, fused = case
    from paper_2411_03171_amd import ffsl
    w = shape(value, L, d, k, B)
    inp, bias = inputs(w, 6)
    Wb, Xb = inp.W.copy(), inp.X.copy()
    inf = np.inf if value == "f32" else 0x7F80
    if where == "weight":
        Wb[77, 3] = inf
    else:
        Xb[B // 2, inp.I[77, 3]] = inf
    inp = synth.dataclasses.replace(inp, W=Wb, X=Xb)
    note("staged infinite %s %s" % (where, case))
    flags = ffsl.FFSL_LOSS_SQHINGE if hinge else 0
    layer = make_gpu_layer(inp, w, bias_values=bias)
    X, off, lab = batch_to_gpu(inp.X, inp.off, inp.lab, w.value)
    if fused:
        _, dX = layer.train_step(X, off, lab, t=1, flags=flags)
    else:
        dX = layer.backward(X, off, lab, flags=flags)
    z, g, dW, db, dXr = plain_grads(w, inp, bias, hinge)
    assert np.isinf(z[:, 77]).any()
    one_plane = fused and k in (32, 64)
    same_with_infinities(dX.cpu().numpy(), dXr, 2e-2 if one_plane else RTOL_F32, "dX")
    if not fused:
        same_with_infinities(layer.dW.cpu().numpy(), dW, RTOL_F32, "dW")
        same_with_infinities(layer.dbias.cpu().numpy(), db, RTOL_F32, "dbias")


@pytest.mark.parametrize("case", [("f32", 30001, 256, 32, 32), ("f32", 4001, 700, 100, 40)], ids=lambda c: "-".join(map(str, c)))
def test_adam_of_the_step_rounds_each_weight_once(torch_cuda, case):
    """The stored weight against float64 Adam on the stored moments, in units of
    its last place: one rounding is uniform in +-1/2, a mean square of 1/12, to
    which the roundings of the update add little where it is far below the weight
    (a product rounded before the sum makes it 1/6).  And an update from zero is
    as exact as divides and a root that each round correctly: the roundings of
    lr m / bc1, v / bc2 (halved by the root), the root, the sum with eps and the
    quotient are 2.25 units of 2^-23 at most, and 1/3 of that in the mean square
    (0.38 when all five are uniform)."""
    torch = torch_cuda
    value, L, d, k, B = case
    w = shape(value, L, d, k, B)
    inp, _ = inputs(w, 11)
    rng = np.random.default_rng(11)
    lr, wd, eps = 1e-4, 1e-3, 1e-8
    for zero in (False, True):
        for t in (3, 1000):
            note("staged Adam %s zero=%s t=%d" % (case, zero, t))
            layer = make_gpu_layer(synth.dataclasses.replace(inp, W=np.zeros_like(inp.W)) if zero else inp, w,
                                   bias_values=np.zeros(L, np.float32), unfused=False)
            layer.m.copy_(torch.from_numpy((rng.standard_normal((L, k)) * 1e-4).astype(np.float32)))
            layer.v.copy_(torch.from_numpy((rng.random((L, k)) * 1e-7).astype(np.float32)))
            W0 = layer.W.double().cpu().numpy()
            X, off, lab = batch_to_gpu(inp.X, inp.off, inp.lab, w.value)
            layer.train_step(X, off, lab, t=t, lr=lr, wd=wd, eps=eps)
            f = lambda x: float(np.float32(x))
            bc1, bc2 = f(1 - f(0.9) ** t), f(1 - f(0.999) ** t)
            m, v = layer.m.double().cpu().numpy(), layer.v.double().cpu().numpy()
            upd = f(lr) * (m / bc1) / (np.sqrt(v / bc2) + f(eps))
            decay = f(np.float32(1) - np.float32(lr) * np.float32(wd))
            ref = W0 * decay - upd
            got = layer.W.double().cpu().numpy()
            if zero:
                rel = np.abs(got - ref) / np.abs(upd)
                assert rel.max() <= 2.25 * 2.0 ** -23
                assert np.sqrt((rel ** 2).mean()) <= 0.75 * 2.0 ** -23
            else:
                far = np.abs(ref) > 64 * np.abs(upd)
                assert far.mean() > 0.05
                ulp = np.spacing(np.abs(ref).astype(np.float32)).astype(np.float64)
                assert (((got - ref) / ulp)[far] ** 2).mean() <= 1.1 / 12


@pytest.mark.parametrize("case", [("bf16", 22003, 150, 100, 1024), ("bf16", 43011, 40, 12, 1024), ("f32", 22003, 128, 70, 1024),
                                  ("f32", 43011, 64, 7, 1024)], ids=lambda c: "-".join(map(str, c)))
def test_fused_step_over_several_slabs(torch_cuda, case):
    """The fused step over two and three slabs and many batch tiles, with three
    planes of g, at fan-ins of four rows and of half a row a unit."""
    torch = torch_cuda
    w = shape(*case)
    inp, bias = inputs(w, 13)
    s, t, lr = 1.0 / w.B, 3, 1e-2
    rng = np.random.default_rng(13)
    m0 = (rng.standard_normal((w.L, w.k)) * 1e-3).astype(np.float32)
    v0 = ((0.5 + rng.random((w.L, w.k))) * 1e-5).astype(np.float32)
    note("staged fused slabs %s" % (case,))
    layer = make_gpu_layer(inp, w, bias_values=bias, unfused=False)
    layer.m.copy_(torch.from_numpy(m0))
    layer.v.copy_(torch.from_numpy(v0))
    X, off, lab = batch_to_gpu(inp.X, inp.off, inp.lab, w.value)
    loss, dX = layer.train_step(X, off, lab, t=t, s=s, lr=lr)
    torch.cuda.synchronize()
    r, Wn, mn, vn, bn, _, _ = adam_reference(w, inp, bias, s, t=t, lr=lr, m0=m0.astype(np.float64), v0=v0.astype(np.float64))
    assert_close(loss.cpu().numpy()[0], r["loss"], RTOL_F32, "loss")
    assert_close(dX.cpu().numpy(), r["dX"], RTOL_F32, "dX")
    assert_close(layer.m.cpu().numpy(), mn, RTOL_F32, "m")
    assert_close(layer.v.cpu().numpy(), vn, 2 * RTOL_F32, "v")   # the square of a gradient
    assert_close(layer.bias.cpu().numpy(), bn, RTOL_F32, "bias")
    Wg = values_f64(from_torch_bits(layer.W, w.value), w.value)
    assert_close(Wg, Wn, RTOL_F32 if w.value == "f32" else 2.0 ** -8, "W")   # bf16: half an ulp


def test_unfused_calls_in_the_least_and_in_a_larger_workspace(torch_cuda):
    """A fan-in-32 layer of one pass: its typed workspace cuts a backward call of
    50000 rows into three slabs, the binding's larger one into one.  Same
    gradients bit for bit, dX up to the order of its sums."""
    import ctypes
    torch = torch_cuda
    from paper_2411_03171_amd import ffsl
    w = shape("bf16", 50000, 128, 32, 64)
    inp, bias = inputs(w, 14)
    X, off, lab = batch_to_gpu(inp.X, inp.off, inp.lab, w.value)
    layer = make_gpu_layer(inp, w, bias_values=bias)
    lib = ffsl.load()
    least = lib.ffsl_workspace_bytes_ex(w.L, w.d, w.k, ffsl.FFSL_BF16, w.B, layer.nnz_max)
    assert layer.workspace.numel() >= least + (16 << 20)
    note("staged in a larger workspace")
    dX = layer.backward(X, off, lab)
    dW, db = layer.dW.clone(), layer.dbias.clone()
    layer.close()
    ptr = ffsl._ptr
    h = ctypes.c_void_p()
    ffsl._check(lib.ffsl_create_layer_ex(ctypes.byref(h), w.L, w.d, w.k, ffsl.FFSL_BF16, layer.idx, ptr(layer.W), ptr(layer.I),
                                         ptr(layer.bias), ptr(layer.m), ptr(layer.v), ptr(layer.bias_m), ptr(layer.bias_v),
                                         ptr(layer.dW), ptr(layer.dbias), ptr(layer.workspace), least, w.B, layer.nnz_max))
    layer._handle = h
    tail = layer.workspace[least:].fill_(7)
    layer.dW.fill_(np.nan)
    note("staged in the least workspace")
    dX2 = layer.backward(X, off, lab)
    assert torch.equal(layer.dW, dW) and torch.equal(layer.dbias, db)
    assert_close(dX2.cpu().numpy(), dX.cpu().numpy(), RTOL_F32, "dX")
    assert bool((tail == 7).all())
