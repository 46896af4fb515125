"""fp32 contractions on the 16-bit matrix unit (operands split into two fp16
halves) against the fp64 oracle, at the edges of their tiles, slots and
launch shapes, and on inputs that one scale does not serve."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
import oracle.layer2d as o2d
import paper_1506_07452_amd as P
import synth
from paper_1506_07452_amd.network import (LayerW, layer2d_backward, layer2d_forward, layer_backward,
                                          layer_forward)
from tests.gpu_util import dev, host, layer_dev, saved_view, say

pytestmark = pytest.mark.gpu

# Splitting loses at most 2^-22 of each operand, 2^-21 of a product, and the sum of n
# products is rounded about n / 32 times, at random: sqrt(n / 32) 2^-24 of the sum of
# magnitudes, 1.2e-6 for the largest n here (12544, 7 x 7 filters over 256 gate-units).
# Both together, 1.7e-6, are carried through the cells of at most 13 planes, each of
# which adds its own (a derivative of h by the h before it is below 1): 2e-5.
TOL = 2e-5
# tanh as 1 - 2 / (e^2a + 1) is off by up to 2^-23 whatever its size: twice in a
# cell, twice in h, over the six directions (one voxel's h is 1e-3 here)
ABS = 6 * 4 * 2.0 ** -23


def close(got, ref):
    return np.abs(got - ref).max() <= TOL * np.abs(ref).max() + ABS


# (N, D, H, W, C, O, K): one pixel; blocks cut by every border; channel counts
# of one slot, several, and a padded last one; slots that end inside a
# K-group; filters whose halo is larger than the plane; every launch shape.
SHAPES = [(1, 1, 1, 1, 1, 32, 3), (1, 5, 9, 11, 6, 16, 3), (2, 3, 7, 40, 17, 16, 5),
          (1, 1, 13, 1, 32, 32, 3), (2, 9, 17, 40, 32, 32, 3), (1, 4, 6, 70, 3, 64, 3),
          (1, 6, 20, 33, 41, 64, 3), (1, 3, 12, 9, 25, 32, 7), (1, 7, 8, 13, 64, 64, 7),
          (1, 3, 5, 4, 9, 16, 1), (1, 3, 120, 130, 8, 32, 3)]


def make(shape, seed):
    N, D, H, W, C, O, K = shape
    return synth.make(synth.Workload("split", N, D, H, W, C, [O], seed=seed, K=K))


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_forward(shape):
    inst = make(shape, 9000 + sum(shape))
    L = inst.layers[0]
    ref = oracle.forward(inst.x, L.wx, L.wh, L.b, want_hd=True, want_saved=True)
    say("split forward", shape)
    x, Ld = dev(inst.x), layer_dev(L)
    h, saved = layer_forward(x, Ld, training=True)
    h2, _ = layer_forward(x, Ld)
    torch.cuda.synchronize()
    assert torch.equal(h, h2)
    assert close(host(h), ref["h"])
    for name in ("hd", "cell", "gates"):
        assert close(saved_view(saved, name, shape[:6]), ref[name]), name


@pytest.mark.parametrize("outlier", [np.inf, -np.inf, 1e30, 1e6], ids=str)
@pytest.mark.parametrize("shape", [(1, 5, 9, 11, 6, 16, 3), (1, 4, 12, 10, 32, 32, 3)],
                         ids=lambda s: "x".join(map(str, s)))
def test_forward_with_an_outlier(shape, outlier):
    """An infinite voxel saturates its neighbours' gates and one far above the
    rest leaves their precision alone, as the fp32 instruction has it."""
    inst = make(shape, 9100 + sum(shape))
    L = inst.layers[0]
    inst.x[0, 2, 4, 5, 1] = outlier
    with np.errstate(over="ignore"):
        ref = oracle.forward(inst.x, L.wx, L.wh, L.b)["h"]
    say("split outlier", shape, outlier)
    h, _ = layer_forward(dev(inst.x), layer_dev(L))
    torch.cuda.synchronize()
    assert np.isfinite(ref).all()
    assert close(host(h), ref)


@pytest.mark.parametrize("want_dx", [True, False], ids=["dx", "no-dx"])
@pytest.mark.parametrize("shape", SHAPES + [(1, 4, 9, 7, 60, 16, 3), (1, 3, 6, 8, 20, 64, 3)],
                         ids=lambda s: "x".join(map(str, s)))
def test_backward(shape, want_dx):
    """Every spread of row tiles over the waves; dL/dh varies by 2^60 from plane to plane,
    so that a scale that does not follow it overflows (what the quiet ones keep is
    test_reverse_keeps_quiet_slices' to see)."""
    inst = make(shape, 9200 + sum(shape))
    L = inst.layers[0]
    dh = synth.upstream_grad(inst.x.shape[:-1] + (shape[5],), 9300 + sum(shape))
    rng = np.random.default_rng(5)
    dh *= np.exp2(rng.integers(-30, 31, size=dh.shape[:2] + (1, 1, 1))).astype(np.float32)
    ref = oracle.backward(inst.x, L.wx, L.wh, L.b, dh)
    say("split backward", shape, want_dx)
    x, Ld = dev(inst.x), layer_dev(L)
    _, saved = layer_forward(x, Ld, training=True)
    dx, dwx, dwh, db = layer_backward(x, Ld, saved, dev(dh), want_dx=want_dx)
    torch.cuda.synchronize()
    check_weights(ref, dwx, dwh, db)
    if dx is not None:
        assert np.abs(host(dx) - ref["dx"]).max() <= TOL * np.abs(ref["dx"]).max()


@pytest.mark.parametrize("shape", [(1, 5, 9, 11, 6, 16, 3), (1, 4, 12, 10, 32, 32, 3)],
                         ids=lambda s: "x".join(map(str, s)))
def test_weight_gradients_with_an_outlier(shape):
    """An input with one value far above the rest keeps the fp32 products: the
    other channels' gradients do not lose theirs."""
    inst = make(shape, 9400 + sum(shape))
    L = inst.layers[0]
    inst.x[0, 2, 4, 5, 1] = 1e12
    dh = synth.upstream_grad(inst.x.shape[:-1] + (shape[5],), 9500 + sum(shape))
    ref = oracle.backward(inst.x, L.wx, L.wh, L.b, dh)
    say("split outlier gradients", shape)
    x, Ld = dev(inst.x), layer_dev(L)
    _, saved = layer_forward(x, Ld, training=True)
    _, dwx, dwh, db = layer_backward(x, Ld, saved, dev(dh))
    torch.cuda.synchronize()
    dwx, rest = host(dwx), [c for c in range(shape[4]) if c != 1]
    assert np.abs(dwx[:, :, rest] - ref["dwx"][:, :, rest]).max() <= TOL * np.abs(ref["dwx"][:, :, rest]).max()
    assert np.abs(dwx - ref["dwx"]).max() <= TOL * np.abs(ref["dwx"]).max()
    for name, got in (("dwh", dwh), ("db", db)):
        assert np.abs(host(got) - ref[name]).max() <= TOL * np.abs(ref[name]).max(), name


@pytest.fixture(params=[0, 3], ids=["whole", "chunked"])
def strips(request):
    P.pyramid_lstm_set_forward_path(request.param)
    try:
        yield
    finally:
        P.pyramid_lstm_set_forward_path(0)


@pytest.mark.parametrize("outlier", [None, np.inf, 1e30], ids=str)
@pytest.mark.parametrize("shape", [(1, 5, 9, 11, 3, 16, 3), (2, 7, 3, 40, 1, 16, 3), (1, 1, 1, 2, 4, 16, 3),
                                   (1, 17, 40, 21, 2, 16, 3)], ids=lambda s: "x".join(map(str, s)))
def test_persistent_forward(shape, outlier, strips):
    """Strips kept whole in LDS and staged by chunks: their tap pairs lie along
    different axes, and the pixel with zero weights may hold an infinity."""
    inst = make(shape, 9600 + sum(shape))
    L = inst.layers[0]
    if outlier is not None:
        inst.x[-1, -1, -1, -1, 0] = outlier
    with np.errstate(over="ignore"):
        ref = oracle.forward(inst.x, L.wx, L.wh, L.b)["h"]
    say("split sweep", shape, outlier)
    h, _ = layer_forward(dev(inst.x), layer_dev(L))
    torch.cuda.synchronize()
    assert close(host(h), ref)


def check_weights(ref, dwx, dwh, db, channels=None):
    """(Against the tensor's largest: a row's own sums may cancel, and what the gate functions
    are off by, 2^-23, is then all that is left.  Rows that are quiet by themselves are
    test_weight_gradients_of_a_closed_gate's.)"""
    for name, got in (("dwx", dwx), ("dwh", dwh), ("db", db)):
        got, want = host(got), ref[name]
        if name == "dwx" and channels is not None:
            got, want = got[:, :, channels], want[:, :, channels]
        assert np.abs(got - want).max() <= TOL * np.abs(want).max(), name


@pytest.mark.parametrize("outlier", [None, 1e12], ids=str)
@pytest.mark.parametrize("path", [0, 2], ids=["whole", "chunked"])
@pytest.mark.parametrize("shape", [(1, 5, 9, 11, 3, 16, 3), (2, 7, 3, 40, 1, 16, 3), (1, 1, 1, 2, 4, 16, 3),
                                   (1, 17, 40, 21, 2, 16, 3)], ids=lambda s: "x".join(map(str, s)))
def test_persistent_weight_gradients(shape, path, outlier):
    """The reverse sweep's own maxima of |dA| scale the products (dL/dh varies by
    2^60 between planes); an input that one scale does not serve keeps fp32."""
    inst = make(shape, 9700 + sum(shape))
    L = inst.layers[0]
    if outlier is not None:
        inst.x[-1, -1, -1, -1, 0] = outlier
    dh = synth.upstream_grad(inst.x.shape[:-1] + (16,), 9800 + sum(shape))
    if outlier is None:
        rng = np.random.default_rng(6)
        dh *= np.exp2(rng.integers(-30, 31, size=dh.shape[:2] + (1, 1, 1))).astype(np.float32)
    ref = oracle.backward(inst.x, L.wx, L.wh, L.b, dh)
    say("split sweep gradients", shape, path, outlier)
    x, Ld = dev(inst.x), layer_dev(L)
    P.pyramid_lstm_set_backward_path(path)
    try:
        _, saved = layer_forward(x, Ld, training=True)
        _, dwx, dwh, db = layer_backward(x, Ld, saved, dev(dh), want_dx=False)
        torch.cuda.synchronize()
    finally:
        P.pyramid_lstm_set_backward_path(0)
    check_weights(ref, dwx, dwh, db)
    if outlier is not None and shape[4] > 1:
        check_weights(ref, dwx, dwh, db, list(range(1, shape[4])))


@pytest.mark.parametrize("outlier", [None, 1e12], ids=str)
@pytest.mark.parametrize("shape", [(1, 1, 1, 1, 1), (2, 33, 40, 1, 3), (1, 9, 129, 4, 5), (3, 70, 6, 17, 7),
                                   (1, 40, 64, 3, 1)], ids=lambda s: "x".join(map(str, s)))
def test_line_weight_gradients(shape, outlier):
    """Lines of one block and several, and those of the reverse line blocks'
    segments over more than one launch."""
    N, H, W, C, K = shape
    x, wx, wh, b = synth.image2d(N, H, W, C, 16, K, 9900 + sum(shape), "f32")
    if outlier is not None:
        x[-1, -1, -1, 0] = outlier
    dh = synth.upstream_grad((N, H, W, 16), 9950 + sum(shape))
    ref = o2d.backward2d(x, wx, wh, b, dh)
    say("split line gradients", shape, outlier)
    xd, L = dev(x), LayerW(dev(wx), dev(wh), dev(b))
    _, saved = layer2d_forward(xd, L, training=True)
    _, dwx, dwh, db = layer2d_backward(xd, L, saved, dev(dh), want_dx=False)
    torch.cuda.synchronize()
    check_weights(ref, dwx, dwh, db)
    if outlier is not None and C > 1:
        check_weights(ref, dwx, dwh, db, list(range(1, C)))


@pytest.mark.parametrize("path", [0, 2], ids=["whole", "chunked"])
@pytest.mark.parametrize("axis", [1, 2, 3], ids=["planes", "rows", "columns"])
def test_persistent_reverse_scales(path, axis):
    """dL/dh that jumps by up to 2^60 from one plane, row or column to the next: a strip's
    scale has to cover what its neighbours hand over, also when they are a step ahead
    (one that is too small overflows; the loudest slice is what this sees)."""
    shape = (1, 19, 40, 52, 2, 16, 3)
    inst = make(shape, 9990 + axis)
    L = inst.layers[0]
    dh = synth.upstream_grad(inst.x.shape[:-1] + (16,), 9995 + axis)
    rng = np.random.default_rng(axis)
    n = [1] * 5
    n[axis] = dh.shape[axis]
    dh *= np.exp2(rng.integers(-30, 31, size=n)).astype(np.float32)
    ref = oracle.backward(inst.x, L.wx, L.wh, L.b, dh)
    say("split reverse scales", path, axis)
    x, Ld = dev(inst.x), layer_dev(L)
    P.pyramid_lstm_set_backward_path(path)
    try:
        _, saved = layer_forward(x, Ld, training=True)
        dx, dwx, dwh, db = layer_backward(x, Ld, saved, dev(dh))
        torch.cuda.synchronize()
    finally:
        P.pyramid_lstm_set_backward_path(0)
    check_weights(ref, dwx, dwh, db)
    assert np.abs(host(dx) - ref["dx"]).max() <= TOL * np.abs(ref["dx"]).max()


def without_neighbours(w):
    """Recurrent filters with their centre tap only: dL/dh of a voxel then reaches the
    voxels of its three axis lines and no others."""
    c = np.zeros_like(w)
    c[..., w.shape[-1] // 2] = w[..., w.shape[-1] // 2]
    if w.ndim == 5:
        c[..., [r for r in range(w.shape[-2]) if r != w.shape[-2] // 2], :] = 0
    return c


def out_of_reach(extents, at, r):
    """Voxels whose dL/dx takes nothing from dL/dh of voxel `at` (at most one coordinate
    within the input filters' radius of it)."""
    near = np.zeros(extents, int)
    for ax, (n, c) in enumerate(zip(extents, at)):
        near += (np.abs(np.arange(n) - c) <= r).reshape([-1 if a == ax else 1 for a in range(len(extents))])
    return near <= len(extents) - 2


STEP_REVERSE = [(1, 5, 9, 11, 6, 16, 3), (1, 5, 12, 10, 32, 32, 3), (1, 5, 8, 9, 16, 64, 3), (1, 5, 8, 9, 40, 64, 3)]
SWEEP_REVERSE = [(1, 5, 9, 11, 3, 16, 3), (1, 19, 40, 52, 2, 16, 3)]    # one strip a direction, several
LOUD = [(s, 0, p) for s in STEP_REVERSE for p in (20, 28, 45, 100)]
LOUD += [(s, path, p) for s in SWEEP_REVERSE for path in (0, 2) for p in (20, 28, 45, 100)]


@pytest.mark.parametrize("shape, path, loud", LOUD, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_reverse_beside_a_loud_voxel(shape, path, loud):
    """Voxels that take nothing from one 2^loud times louder keep their precision, though
    its block or strip has one scale: the residual half reaches as far down as the first,
    and where that is not enough the block keeps fp32."""
    inst = make(shape, 9100 + sum(shape))
    L = inst.layers[0]
    L.wh = without_neighbours(L.wh)
    dh = synth.upstream_grad(inst.x.shape[:-1] + (shape[5],), 77)
    dh[0, 2, 4, 5] *= 2.0 ** loud
    ref = oracle.backward(inst.x, L.wx, L.wh, L.b, dh)["dx"][0]
    quiet = out_of_reach(shape[1:4], (2, 4, 5), 1)
    say("split loud voxel", shape, path, loud)
    x, Ld = dev(inst.x), layer_dev(L)
    P.pyramid_lstm_set_backward_path(path)
    try:
        _, saved = layer_forward(x, Ld, training=True)
        dx, _, _, _ = layer_backward(x, Ld, saved, dev(dh))
        torch.cuda.synchronize()
    finally:
        P.pyramid_lstm_set_backward_path(0)
    assert np.abs(host(dx)[0][quiet] - ref[quiet]).max() <= TOL * np.abs(ref[quiet]).max()


@pytest.mark.parametrize("which, at", [("wh", (0, 3, 1)), ("wx", (2, 18, 2))], ids=["wh", "wx"])
@pytest.mark.parametrize("shape, path", [(s, 0) for s in STEP_REVERSE] + [(s, p) for s in SWEEP_REVERSE for p in (0, 2)],
                         ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_reverse_with_an_outlier_weight(shape, path, which, at):
    """A weight of 1e30 shuts its gate, whose gradient is 0: the other weights of that unit
    or channel keep theirs."""
    inst = make(shape, 9100 + sum(shape))
    L = inst.layers[0]
    getattr(L, which)[at[:2] + (min(at[2], getattr(L, which).shape[2] - 1), 1, 1)] = 1e30
    dh = synth.upstream_grad(inst.x.shape[:-1] + (shape[5],), 77)
    with np.errstate(all="ignore"):
        ref = oracle.backward(inst.x, L.wx, L.wh, L.b, dh)
    say("split reverse outlier weight", shape, path, which)
    x, Ld = dev(inst.x), layer_dev(L)
    P.pyramid_lstm_set_backward_path(path)
    try:
        _, saved = layer_forward(x, Ld, training=True)
        dx, dwx, dwh, db = layer_backward(x, Ld, saved, dev(dh))
        torch.cuda.synchronize()
    finally:
        P.pyramid_lstm_set_backward_path(0)
    check_weights(ref, dwx, dwh, db)
    dx, want = host(dx), ref["dx"]
    for c in range(shape[4]):
        assert np.abs(dx[..., c] - want[..., c]).max() <= TOL * np.abs(want[..., c]).max(), c


@pytest.mark.parametrize("shape", [(1, 1, 9, 11, 6, 16, 3), (1, 1, 9, 11, 3, 16, 3)], ids=lambda s: "x".join(map(str, s)))
def test_weight_gradients_of_an_infinite_dh(shape):
    """Rows of a gate with an infinite gradient are infinite where 64 bits have them so (a
    residual of infinity makes them NaN)."""
    inst = make(shape, 9100 + sum(shape))
    L = inst.layers[0]
    L.wh[:] = 0
    dh = synth.upstream_grad(inst.x.shape[:-1] + (shape[5],), 79)
    dh[0, 0, 4, 5, 7] = np.inf
    with np.errstate(all="ignore"):
        ref = oracle.backward(inst.x, L.wx, L.wh, L.b, dh)
    x, Ld = dev(inst.x), layer_dev(L)
    say("split infinite dh", shape)
    _, saved = layer_forward(x, Ld, training=True)
    _, dwx, _, db = layer_backward(x, Ld, saved, dev(dh))
    torch.cuda.synchronize()
    for got, want in ((dwx, ref["dwx"]), (db, ref["db"])):
        assert np.isinf(want).any()
        assert (host(got)[np.isinf(want)] == want[np.isinf(want)]).all()


@pytest.mark.parametrize("loud", [20, 28, 45, 100])
@pytest.mark.parametrize("shape", [(1, 21, 30, 3, 3), (1, 12, 70, 1, 5), (2, 40, 9, 6, 3)],
                         ids=lambda s: "x".join(map(str, s)))
def test_line_reverse_beside_a_loud_pixel(shape, loud):
    N, H, W, C, K = shape
    x, wx, wh, b = synth.image2d(N, H, W, C, 16, K, 9900 + sum(shape), "f32")
    wh = without_neighbours(wh)
    dh = synth.upstream_grad((N, H, W, 16), 78)
    dh[0, 5, 4] *= 2.0 ** loud
    ref = o2d.backward2d(x, wx, wh, b, dh)["dx"][0]
    quiet = out_of_reach((H, W), (5, 4), K // 2)
    say("split loud pixel", shape, loud)
    xd, L = dev(x), LayerW(dev(wx), dev(wh), dev(b))
    _, saved = layer2d_forward(xd, L, training=True)
    dx, _, _, _ = layer2d_backward(xd, L, saved, dev(dh))
    torch.cuda.synchronize()
    assert np.abs(host(dx)[0][quiet] - ref[quiet]).max() <= TOL * np.abs(ref[quiet]).max()


def closed_gate_error(ref, got, O, unit):
    """Largest error of the rows of an input gate relative to the row's own largest."""
    worst = 0.0
    for name in ("dwx", "dwh"):
        r, g = ref[name][:, unit].reshape(6, -1), host(got[name])[:, unit].reshape(6, -1)
        worst = max(worst, (np.abs(g - r).max(1) / np.abs(r).max(1)).max())
    return worst


@pytest.mark.parametrize("bias", [-18, -22, -30, -60])
@pytest.mark.parametrize("shape", [(1, 5, 9, 11, 6, 16, 3), (1, 4, 12, 10, 32, 32, 3), (1, 5, 9, 11, 3, 16, 3)],
                         ids=lambda s: "x".join(map(str, s)))
def test_weight_gradients_of_a_closed_gate(shape, bias):
    """An input gate shut by its bias has gradients e^bias of the others'; its rows of dW
    keep their precision beside theirs, in fp32 where one scale does not serve both."""
    inst = make(shape, 9100 + sum(shape))
    L = inst.layers[0]
    L.b[:, 5] = bias
    dh = synth.upstream_grad(inst.x.shape[:-1] + (shape[5],), 79)
    ref = oracle.backward(inst.x, L.wx, L.wh, L.b, dh)
    say("split closed gate", shape, bias)
    x, Ld = dev(inst.x), layer_dev(L)
    _, saved = layer_forward(x, Ld, training=True)
    _, dwx, dwh, _ = layer_backward(x, Ld, saved, dev(dh))
    torch.cuda.synchronize()
    assert closed_gate_error(ref, {"dwx": dwx, "dwh": dwh}, shape[5], 5) <= TOL


FORWARD_SHAPES = [(1, 12, 9, 11, 6, 16, 3), (1, 8, 12, 10, 32, 32, 3), (1, 12, 20, 11, 3, 16, 3)]


@pytest.mark.parametrize("zero_rows", [False, True], ids=["dense", "zero-rows"])
@pytest.mark.parametrize("big", [1e7, 1e9, 1e12, 1e14], ids=str)
@pytest.mark.parametrize("shape", FORWARD_SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_forward_of_a_masked_volume(shape, big, zero_rows, strips):
    """Zeros beside large values: the recurrence of the empty half keeps its weights,
    whatever scale x asks for, and a gate row without weights adds nothing.  An operand
    is off by what changes its product by at most 2^-29, over n products and six
    directions."""
    inst = make(shape, 9100 + sum(shape))
    L = inst.layers[0]
    inst.x[:, :, :, shape[3] // 2:] = 0
    inst.x *= big
    inst.x[0, 0, 0, -1, 0] = 1.0
    if zero_rows:
        L.wx[:, 5], L.wh[:, 5] = 0, 0
    with np.errstate(over="ignore"):
        ref = oracle.forward(inst.x, L.wx, L.wh, L.b)["h"]
    say("split masked", shape, big, zero_rows)
    h, _ = layer_forward(dev(inst.x), layer_dev(L))
    torch.cuda.synchronize()
    n = 9 * (shape[4] + shape[5])
    assert np.abs(host(h) - ref).max() <= 6 * 2 * n * 2.0 ** -29 + ABS


@pytest.mark.parametrize("which, value", [("wx", np.inf), ("wx", -np.inf), ("wx", 1e30), ("wh", np.inf), ("wh", -np.inf),
                                          ("wh", 1e30)], ids=lambda v: str(v))
@pytest.mark.parametrize("shape", FORWARD_SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_forward_with_an_outlier_weight(shape, which, value, strips):
    """An infinite weight saturates its gate (0 times it is NaN in the persistent sweep,
    whose first plane multiplies by h = 0), and one of 1e30 leaves the others alone."""
    if which == "wh" and np.isinf(value) and shape[4] <= 4:
        pytest.skip("the persistent sweep multiplies by h = 0")
    inst = make(shape, 9100 + sum(shape))
    L = inst.layers[0]
    getattr(L, which)[0, 3, 1, 1, 1] = value
    with np.errstate(all="ignore"):
        ref = oracle.forward(inst.x, L.wx, L.wh, L.b)["h"]
    say("split outlier weight", shape, which, value)
    h, _ = layer_forward(dev(inst.x), layer_dev(L))
    torch.cuda.synchronize()
    assert np.isfinite(ref).all()
    assert close(host(h), ref)


@pytest.mark.parametrize("value", [np.inf, -np.inf, 1e12], ids=str)
@pytest.mark.parametrize("shape", [(1, 20, 70, 2, 3), (2, 35, 33, 5, 7)], ids=lambda s: "x".join(map(str, s)))
def test_line_forward_with_an_outlier_weight(shape, value):
    """As above for the 2D line blocks, over more than one launch; the volume with D = 1 that
    computes the layer has no product with h before the first line."""
    N, H, W, C, K = shape
    x, wx, wh, b = synth.image2d(N, H, W, C, 16, K, 9910 + sum(shape), "f32")
    wh[:, 3, 1, K // 2] = value
    with np.errstate(all="ignore"):
        ref = o2d.forward2d_via_volume(x, wx, wh, b)
    say("split outlier line weight", shape, value)
    h, _ = layer2d_forward(dev(x), LayerW(dev(wx), dev(wh), dev(b)))
    torch.cuda.synchronize()
    assert np.isfinite(ref).all()
    assert close(host(h), ref)


@pytest.mark.parametrize("which, at", [("wh", (0, 3, 1)), ("wx", (2, 18, 0))], ids=["wh", "wx"])
@pytest.mark.parametrize("shape", [(1, 21, 30, 3, 3), (2, 40, 9, 6, 5)], ids=lambda s: "x".join(map(str, s)))
def test_line_reverse_with_an_outlier_weight(shape, which, at):
    N, H, W, C, K = shape
    x, wx, wh, b = synth.image2d(N, H, W, C, 16, K, 9920 + sum(shape), "f32")
    {"wx": wx, "wh": wh}[which][at + (K // 2,)] = 1e30
    dh = synth.upstream_grad((N, H, W, 16), 78)
    with np.errstate(all="ignore"):
        ref = o2d.backward2d(x, wx, wh, b, dh)
    say("split line reverse outlier weight", shape, which)
    xd, L = dev(x), LayerW(dev(wx), dev(wh), dev(b))
    _, saved = layer2d_forward(xd, L, training=True)
    dx, dwx, dwh, db = layer2d_backward(xd, L, saved, dev(dh))
    torch.cuda.synchronize()
    check_weights(ref, dwx, dwh, db)
    assert np.abs(host(dx) - ref["dx"]).max() <= TOL * np.abs(ref["dx"]).max()


@pytest.mark.parametrize("axis", [0, 1, 2], ids=["planes", "rows", "columns"])
@pytest.mark.parametrize("channels, units, path", [(6, 16, 0), (32, 32, 0), (20, 64, 0), (3, 16, 0), (3, 16, 2)])
def test_reverse_keeps_quiet_slices(channels, units, path, axis):
    """Groups of three slices of dL/dh up to 2^50 apart that nothing leaks between: the
    recurrence along the axis is off (no weights, shut forget gates), the others have their
    centre tap only, and the input filters reach one slice.  The middle one of each group is
    compared with its own largest: a scale common to all would leave the quiet ones at
    2^-50 of the loud ones, with no digit of their own."""
    shape = (1, 12, 12, 15, channels, units, 3)
    inst = make(shape, 9980 + axis + units)
    L = inst.layers[0]
    L.wh = without_neighbours(L.wh)
    L.wh[2 * axis:2 * axis + 2] = 0
    L.b[2 * axis:2 * axis + 2, units:2 * units] = -60
    dh = synth.upstream_grad(inst.x.shape[:-1] + (units,), 9985 + axis)
    steps = np.array([0, -50, 0, -25, -50])[np.arange(shape[1 + axis]) // 3 % 5]
    dh *= np.exp2(steps).astype(np.float32).reshape([-1 if a == 1 + axis else 1 for a in range(5)])
    ref = oracle.backward(inst.x, L.wx, L.wh, L.b, dh)["dx"]
    say("split quiet slices", shape, path, axis)
    x, Ld = dev(inst.x), layer_dev(L)
    P.pyramid_lstm_set_backward_path(path)
    try:
        _, saved = layer_forward(x, Ld, training=True)
        dx, _, _, _ = layer_backward(x, Ld, saved, dev(dh))
        torch.cuda.synchronize()
    finally:
        P.pyramid_lstm_set_backward_path(0)
    dx, top = np.moveaxis(host(dx), 1 + axis, 0), []
    for k, want in enumerate(np.moveaxis(ref, 1 + axis, 0)):
        if k % 3 == 1:
            top.append(np.abs(want).max())
            assert np.abs(dx[k] - want).max() <= TOL * top[-1], (k, np.abs(dx[k] - want).max() / top[-1])
    assert min(top) < 2.0 ** -40 * max(top)
