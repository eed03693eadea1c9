"""GPU parity of the recurrence kernels over the hidden sizes and batch sizes
they are built for, against the fp64 oracle: every instantiation of the
XCD-local kernels (one and two blocks of sequences per XCD, whole and partial
blocks, several rounds of sequences), variable lengths and carried state."""

import numpy as np
import pytest

import oracle
from paper_1904_10584_amd import binding as am
from tests.gpu_util import gpu_forward_backward, oracle_forward_backward, say
from tests.test_gpu_model import BF16_TOL, F32_TOL, _check, _problem

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def default_paths(monkeypatch):
    for k in ("AM_STEP_KERNELS", "AM_XCD_FENCED", "AM_RECURRENCE", "AM_XCD_BLOCKS"):
        monkeypatch.delenv(k, raising=False)


# (hidden, sequences): sequences 33 fill two blocks and start a third, 150 use
# two blocks per XCD (up to hidden 768) or two rounds, 270 and 400 more rounds
SHAPES = [(64, 33), (64, 270), (128, 150), (128, 1000), (192, 33), (192, 150), (256, 33), (256, 150), (320, 33), (320, 150),
          (384, 33), (384, 150), (448, 33), (448, 150), (512, 33), (512, 270), (576, 33), (576, 150),
          (640, 33), (640, 150), (704, 33), (704, 150), (768, 33), (768, 270), (832, 33), (896, 33),
          (960, 150), (1024, 33), (1024, 400)]


@pytest.mark.parametrize("hidden,B", SHAPES)
def test_bf16_recurrence_shapes(hidden, B):
    dims = oracle.ModelDims(2, 40, hidden, 72)
    T = 5
    lengths = np.sort(np.random.default_rng(hidden + B).integers(0, T + 1, B))[::-1].astype(np.int32)
    lengths[0] = T
    m = am.Model(dims.layers, dims.input_dim, dims.hidden, dims.classes, am.BF16)
    say(f"recurrence shape H={hidden} B={B} path {am.recurrence_path(m, T, B, True)}")
    master, x, idx, prob, h0, c0 = _problem(dims, T, B, 6, 0.98, lengths, seed=23, state=True)
    got = gpu_forward_backward(m, master, x, T, B, idx, prob, lengths, h0, c0, want_state=True)
    ref = oracle_forward_backward(dims, master, x, T, B, idx, prob, lengths, h0, c0, bf16=True)
    _check(got, ref, dims, BF16_TOL, state=True)


# the same on the XCD-local kernels alone, one layer after another (few sequences
# would go through all layers in one launch, 64 cells through the solo kernels)
@pytest.mark.parametrize("hidden,B", SHAPES + [(128, 33), (256, 270), (448, 128), (640, 128), (704, 128)])
def test_bf16_recurrence_shapes_layer_after_layer(hidden, B, monkeypatch):
    monkeypatch.setenv("AM_RECURRENCE", "xcd")
    dims = oracle.ModelDims(2, 40, hidden, 72)
    rounds = -(-B // (256 if hidden <= 768 else 128))
    T = 5 if rounds == 1 else 4 * rounds + 1
    lengths = np.sort(np.random.default_rng(hidden + B).integers(0, T + 1, B))[::-1].astype(np.int32)
    lengths[0] = T
    m = am.Model(dims.layers, dims.input_dim, dims.hidden, dims.classes, am.BF16)
    say(f"recurrence shape, layer after layer H={hidden} B={B} T={T}")
    for fwd in (True, False):
        assert am.recurrence_path(m, T, B, True, fwd) == am.PATH_XCD
    master, x, idx, prob, h0, c0 = _problem(dims, T, B, 6, 0.98, lengths, seed=23, state=True)
    am.profile_begin([am.KERNEL_CLASSES.index(k) for k in ("lstm_fwd", "lstm_bwd")])
    try:
        got = gpu_forward_backward(m, master, x, T, B, idx, prob, lengths, h0, c0, want_state=True)
    finally:
        am.profile_end()
    for k in ("lstm_fwd", "lstm_bwd"):  # (one record a layer, whatever its rounds)
        assert am.profile_get(am.KERNEL_CLASSES.index(k))["launches"] == dims.layers
    ref = oracle_forward_backward(dims, master, x, T, B, idx, prob, lengths, h0, c0, bf16=True)
    _check(got, ref, dims, BF16_TOL, state=True)


# one workgroup per 16 sequences: every width it is built for, a lone sequence,
# a whole workgroup, one more; one step, fewer and more steps than the operand
# ring has slots
@pytest.mark.parametrize("dtype,hidden", [("bf16", h) for h in range(16, 129, 16)] +
                         [("f32", h) for h in range(16, 97, 16)])
@pytest.mark.parametrize("B,T,varlen", [(1, 1, False), (16, 3, True), (17, 11, True), (40, 4, False)])
def test_narrow_layers(dtype, hidden, B, T, varlen):
    bf16 = dtype == "bf16"
    dims = oracle.ModelDims(2, 24, hidden, 40)
    lengths = None
    if varlen:
        lengths = np.sort(np.random.default_rng(hidden + B).integers(0, T + 1, B))[::-1].astype(np.int32)
        lengths[0] = T
    m = am.Model(dims.layers, dims.input_dim, dims.hidden, dims.classes, am.BF16 if bf16 else am.F32)
    if hidden < 128:
        assert am.recurrence_path(m, T, B, varlen) == am.PATH_SOLO
    say(f"narrow layer {dtype} H={hidden} B={B} T={T} varlen={varlen}")
    master, x, idx, prob, h0, c0 = _problem(dims, T, B, 6, 0.98, lengths, seed=37, state=True)
    got = gpu_forward_backward(m, master, x, T, B, idx, prob, lengths, h0, c0, want_state=True)
    ref = oracle_forward_backward(dims, master, x, T, B, idx, prob, lengths, h0, c0, bf16=bf16)
    _check(got, ref, dims, BF16_TOL if bf16 else F32_TOL, state=True)


@pytest.mark.parametrize("hidden,B", [(256, 20), (512, 48), (704, 140), (1024, 130)])
def test_bf16_recurrence_shapes_run_repeatedly(hidden, B):
    # many steps on warm caches, several passes on one workspace: every pass
    # gives the first one's bits, and no step barrier runs out
    dims = oracle.ModelDims(1, 40, hidden, 72)
    T = 60
    m = am.Model(dims.layers, dims.input_dim, dims.hidden, dims.classes, am.BF16)
    say(f"recurrence repeat H={hidden} B={B}")
    master, x, idx, prob, _, _ = _problem(dims, T, B, 6, 0.98, seed=29)
    first = gpu_forward_backward(m, master, x, T, B, idx, prob)
    for _ in range(3):
        again = gpu_forward_backward(m, master, x, T, B, idx, prob)
        for k in ("logits", "dlogits", "grads"):
            np.testing.assert_array_equal(again[k].view(np.uint32), first[k].view(np.uint32))


# the forward exchange within an XCD (rows polled in a ring) against the fenced
# one (flags), over enough steps that the ring's slots turn over and members
# drift: the same bits.  Odd and even numbers of 128-byte lines per row, one and
# two blocks per XCD, sequences that end at different steps
@pytest.mark.parametrize("hidden,B", [(64, 9), (192, 150), (320, 40), (512, 140), (576, 17), (768, 128), (768, 200),
                                      (832, 5), (1024, 300)])
def test_ring_exchange_equals_flags(hidden, B, monkeypatch):
    dims = oracle.ModelDims(1, 24, hidden, 40)
    T = 180
    lengths = np.sort(np.random.default_rng(hidden + B).integers(T // 3, T + 1, B))[::-1].astype(np.int32)
    lengths[0] = T
    m = am.Model(dims.layers, dims.input_dim, dims.hidden, dims.classes, am.BF16)
    say(f"ring exchange H={hidden} B={B}")
    monkeypatch.setenv("AM_RECURRENCE", "xcd")
    master, x, idx, prob, h0, c0 = _problem(dims, T, B, 6, 0.98, lengths, seed=59, state=True)
    got = gpu_forward_backward(m, master, x, T, B, idx, prob, lengths, h0, c0, want_state=True)
    monkeypatch.setenv("AM_XCD_FENCED", "1")
    ref = gpu_forward_backward(m, master, x, T, B, idx, prob, lengths, h0, c0, want_state=True)
    for k in ref:
        np.testing.assert_array_equal(np.asarray(got[k]), np.asarray(ref[k]))


# every layer in one launch: each instantiation, an XCD or half of one per
# (layer, block), up to every slot taken; more blocks than slots (the last) go
# layer by layer
@pytest.mark.parametrize("layers,hidden,B,T", [
    (2, 128, 20, 9), (8, 128, 32, 4), (3, 192, 33, 5), (4, 256, 17, 6), (2, 256, 128, 5), (2, 320, 16, 7),
    (5, 320, 48, 4), (3, 384, 16, 5), (3, 384, 70, 5), (2, 448, 60, 4), (3, 448, 80, 4), (4, 512, 32, 5),
    (3, 512, 48, 11), (2, 576, 16, 5), (3, 640, 20, 5), (4, 704, 32, 4), (5, 768, 12, 9), (8, 768, 1, 3),
    (2, 768, 3, 1), (5, 512, 64, 3)])
@pytest.mark.parametrize("varlen", [False, True])
def test_layers_in_one_launch(layers, hidden, B, T, varlen):
    dims = oracle.ModelDims(layers, 40, hidden, 72)
    lengths = None
    if varlen:
        lengths = np.sort(np.random.default_rng(hidden + B).integers(0, T + 1, B))[::-1].astype(np.int32)
        lengths[0] = T
    m = am.Model(dims.layers, dims.input_dim, dims.hidden, dims.classes, am.BF16)
    say(f"layers in one launch L={layers} H={hidden} B={B} T={T} varlen={varlen}")
    master, x, idx, prob, h0, c0 = _problem(dims, T, B, 6, 0.98, lengths, seed=43, state=varlen)
    got = gpu_forward_backward(m, master, x, T, B, idx, prob, lengths, h0, c0, want_state=True)
    ref = oracle_forward_backward(dims, master, x, T, B, idx, prob, lengths, h0, c0, bf16=True)
    _check(got, ref, dims, BF16_TOL, state=True)


# the same shapes: the query says so, and the pass is one launch (the last one's
# is one a layer)
@pytest.mark.parametrize("layers,hidden,B,T", [
    (2, 128, 20, 9), (8, 128, 32, 4), (3, 192, 33, 5), (4, 256, 17, 6), (2, 256, 128, 5), (2, 320, 16, 7),
    (5, 320, 48, 4), (3, 384, 16, 5), (3, 384, 70, 5), (2, 448, 60, 4), (3, 448, 80, 4), (4, 512, 32, 5),
    (3, 512, 48, 11), (2, 576, 16, 5), (3, 640, 20, 5), (4, 704, 32, 4), (5, 768, 12, 9), (8, 768, 1, 3),
    (2, 768, 3, 1), (5, 512, 64, 3)])
def test_layers_in_one_launch_taken(layers, hidden, B, T):
    piped = (layers, hidden, B) != (5, 512, 64)
    m = am.Model(layers, 40, hidden, 72, am.BF16)
    say(f"layers in one launch, launches L={layers} H={hidden} B={B} T={T}")
    assert am.recurrence_path(m, T, B) == (am.PATH_PIPE if piped else am.PATH_XCD)
    assert am.recurrence_path(m, T, B, False, False) == am.PATH_XCD
    master, x, idx, prob, _, _ = _problem(oracle.ModelDims(layers, 40, hidden, 72), T, B, 6, 0.98, seed=43)
    am.profile_begin([am.KERNEL_CLASSES.index("lstm_fwd")])
    try:
        gpu_forward_backward(m, master, x, T, B, idx, prob)
    finally:
        am.profile_end()
    assert am.profile_get(am.KERNEL_CLASSES.index("lstm_fwd"))["launches"] == (1 if piped else layers)


@pytest.mark.parametrize("layers,hidden,B,T,fenced", [(5, 768, 12, 150, False), (3, 512, 48, 150, False),
                                                      (5, 256, 40, 150, False), (4, 384, 30, 40, True)])
def test_layers_in_one_launch_run_repeatedly(layers, hidden, B, T, fenced, monkeypatch):
    # the layers follow one another over many steps, on one workspace, always
    # with the same bits, and as close to one layer after another as two
    # summation orders of the projections are
    if fenced:
        monkeypatch.setenv("AM_XCD_FENCED", "1")
    dims = oracle.ModelDims(layers, 40, hidden, 72)
    m = am.Model(dims.layers, dims.input_dim, dims.hidden, dims.classes, am.BF16)
    say(f"layers in one launch, repeated L={layers} H={hidden} B={B}")
    master, x, idx, prob, _, _ = _problem(dims, T, B, 6, 0.98, seed=47)
    first = gpu_forward_backward(m, master, x, T, B, idx, prob)
    for _ in range(3):
        again = gpu_forward_backward(m, master, x, T, B, idx, prob)
        for k in ("logits", "dlogits", "grads"):
            np.testing.assert_array_equal(again[k].view(np.uint32), first[k].view(np.uint32))
    monkeypatch.setenv("AM_RECURRENCE", "xcd")
    one = gpu_forward_backward(m, master, x, T, B, idx, prob)
    for k in ("logits", "grads"):
        a, b = first[k].astype(np.float64), one[k].astype(np.float64)
        assert np.linalg.norm(a - b) <= 1e-2 * np.linalg.norm(b)


@pytest.mark.parametrize("layers,hidden,B,T,varlen", [
    (5, 768, 12, 32, False), (4, 704, 32, 20, True), (3, 640, 20, 20, False), (2, 576, 16, 9, False),
    (3, 512, 48, 40, True), (2, 448, 60, 20, False), (3, 384, 70, 20, True), (2, 320, 16, 20, False),
    (5, 256, 40, 30, False), (3, 192, 33, 12, True), (8, 128, 32, 9, False)])
def test_layers_in_one_launch_give_the_bits_of_layer_after_layer(layers, hidden, B, T, varlen, monkeypatch):
    # each launch's shape: the layers above the first get the same projections
    # to the last bit, whichever kernel makes them
    dims = oracle.ModelDims(layers, 40, hidden, 72)
    lengths = None
    if varlen:
        lengths = np.sort(np.random.default_rng(hidden + B).integers(0, T + 1, B))[::-1].astype(np.int32)
        lengths[0] = T
    m = am.Model(dims.layers, dims.input_dim, dims.hidden, dims.classes, am.BF16)
    say(f"one launch against layer after layer L={layers} H={hidden} B={B} T={T} varlen={varlen}")
    assert am.recurrence_path(m, T, B, varlen) == am.PATH_PIPE
    master, x, idx, prob, h0, c0 = _problem(dims, T, B, 6, 0.98, lengths, seed=61, state=True)
    got = gpu_forward_backward(m, master, x, T, B, idx, prob, lengths, h0, c0, want_state=True)
    monkeypatch.setenv("AM_RECURRENCE", "xcd")
    ref = gpu_forward_backward(m, master, x, T, B, idx, prob, lengths, h0, c0, want_state=True)
    for k in ref:
        np.testing.assert_array_equal(np.asarray(got[k]).view(np.uint32) if k != "loss" else got[k],
                                      np.asarray(ref[k]).view(np.uint32) if k != "loss" else ref[k])


@pytest.mark.parametrize("hidden,B,longest", [(192, 9, 40), (320, 150, 900), (768, 128, 25), (256, 1000, 30),
                                              (1024, 300, 13), (384, 492, 8)])
def test_active_sequences_read_or_walked(hidden, B, longest, monkeypatch):
    # up to 1024 steps the kernels read each step's active sequences, beyond they
    # walk the sorted lengths; T beyond the longest sequence changes nothing else
    monkeypatch.setenv("AM_RECURRENCE", "xcd")
    dims = oracle.ModelDims(1, 24, hidden, 40)
    lengths = np.sort(np.random.default_rng(hidden + B).integers(0, longest + 1, B))[::-1].astype(np.int32)
    lengths[0] = longest
    m = am.Model(dims.layers, dims.input_dim, dims.hidden, dims.classes, am.BF16)
    say(f"active sequences H={hidden} B={B} longest={longest}")
    assert all(am.recurrence_path(m, T, B, True) == am.PATH_XCD for T in (longest, 1100))
    master, x, idx, prob, h0, c0 = _problem(dims, longest, B, 6, 0.98, lengths, seed=67, state=True)
    got = gpu_forward_backward(m, master, x, longest, B, idx, prob, lengths, h0, c0, want_state=True)
    ref = gpu_forward_backward(m, master, x, 1100, B, idx, prob, lengths, h0, c0, want_state=True)
    for k in ref:
        np.testing.assert_array_equal(np.asarray(got[k]), np.asarray(ref[k]))
