"""GPU parity of the one-launch backward step (product and cell) of wide
layers against the fp64 oracle: whole and partial tiles of rows and units,
sequences that end at different steps (row tiles without a next step, steps
that fall back to the split product), carried state."""

import numpy as np
import pytest

import oracle
from paper_1904_10584_amd import binding as am
from tests.gpu_util import gpu_forward_backward, oracle_forward_backward, say
from tests.test_gpu_model import BF16_TOL, _check, _problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hidden,B,varlen", [(1536, 256, False), (1056, 385, False), (1088, 512, True),
                                             (1184, 330, True), (2080, 192, False)])
def test_fused_backward_step(hidden, B, varlen, monkeypatch):
    monkeypatch.setenv("AM_RECURRENCE", "step")
    dims = oracle.ModelDims(1, 24, hidden, 40)
    T = 4
    lengths = None
    if varlen:
        lengths = np.sort(np.random.default_rng(hidden).integers(0, T + 1, B))[::-1].astype(np.int32)
        lengths[0] = T
    m = am.Model(1, 24, hidden, 40, am.BF16)
    say(f"fused backward step H={hidden} B={B} varlen={varlen}")
    master, x, idx, prob, h0, c0 = _problem(dims, T, B, 4, 0.98, lengths, seed=53, state=True)
    got = gpu_forward_backward(m, master, x, T, B, idx, prob, lengths, h0, c0, want_state=True)
    ref = oracle_forward_backward(dims, master, x, T, B, idx, prob, lengths, h0, c0, bf16=True)
    _check(got, ref, dims, BF16_TOL, state=True)


def _backward_launches(m, T, B, lengths=None):
    """Timed launches of one backward pass's recurrence: one a step where it is
    fused, else the product (but for the last step's) and the cell."""
    dims = oracle.ModelDims(m.layers, m.input_dim, m.hidden, m.classes)
    prob_ = _problem(dims, T, B, 4, 0.98, lengths, seed=71)
    am.profile_begin([am.KERNEL_CLASSES.index("lstm_bwd")])
    try:
        got = gpu_forward_backward(m, *prob_[:2], T, B, *prob_[2:4], lengths)
    finally:
        am.profile_end()
    return am.profile_get(am.KERNEL_CLASSES.index("lstm_bwd"))["launches"], got, prob_


# enough steps of a covered shape are fused, every other pass is split: fewer
# steps than pay for the transpose (one has no product at all), more than 256
# tiles, fewer than 128, widths beyond 2048
@pytest.mark.parametrize("hidden,B,T,fused", [
    (1536, 256, 5, True), (1056, 385, 4, True), (768, 1024, 3, True), (2048, 192, 6, True),
    (1536, 256, 4, False), (1536, 512, 1, False), (1056, 385, 3, False), (768, 1024, 2, False),
    (1536, 576, 6, False), (2048, 384, 6, False), (1536, 192, 6, False), (2080, 192, 8, False)])
def test_backward_step_route(hidden, B, T, fused, monkeypatch):
    monkeypatch.setenv("AM_RECURRENCE", "step")
    m = am.Model(1, 24, hidden, 40, am.BF16)
    say(f"backward step route H={hidden} B={B} T={T} fused={fused}")
    assert _backward_launches(m, T, B)[0] == (T if fused else 2 * T - 1)


# the shapes above at lengths that fuse, against the oracle; steps of a ragged
# batch that leave the covered tiles are split
@pytest.mark.parametrize("hidden,B,T,varlen,launches", [(1536, 256, 6, False, 6), (1056, 385, 5, False, 5),
                                                        (1088, 512, 12, True, None), (768, 1024, 4, False, 4)])
def test_fused_backward_steps_taken(hidden, B, T, varlen, launches, monkeypatch):
    monkeypatch.setenv("AM_RECURRENCE", "step")
    lengths = None
    if varlen:
        lengths = np.sort(np.random.default_rng(hidden).integers(T // 2, T + 1, B))[::-1].astype(np.int32)
        lengths[0] = T
        tiles = -(-hidden // 48) * -(-np.array([(lengths > t).sum() for t in range(T)]) // 64)
        on = (tiles >= 128) & (tiles <= 256)
        assert on.any() and not on.all()
        launches = int(on.sum() + 2 * (~on).sum() - (0 if on[-1] else 1))
    m = am.Model(1, 24, hidden, 40, am.BF16)
    say(f"fused backward steps H={hidden} B={B} T={T} varlen={varlen}")
    n, got, (master, x, idx, prob, _, _) = _backward_launches(m, T, B, lengths)
    assert n == launches
    dims = oracle.ModelDims(1, 24, hidden, 40)
    ref = oracle_forward_backward(dims, master, x, T, B, idx, prob, lengths, bf16=True)
    _check(got, ref, dims, BF16_TOL)
