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
