"""GPU parity of the fp32 products at sizes that take each tile edge (128, 64
and 32 rows) with remainders, through an fp32 model's forward and backward
against the fp64 oracle (two-source weight gradients with row sums and k-splits
among them)."""

import pytest

import oracle
from paper_1904_10584_amd import binding as am
from tests.gpu_util import gpu_forward_backward, oracle_forward_backward, say
from tests.test_gpu_model import F32_TOL, _check, _problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layers,input_dim,hidden,classes,T,B", [
    (1, 4, 16, 4, 1, 1),          # one partial tile each
    (2, 36, 48, 100, 9, 13),      # a few small tiles, ragged in every direction
    (2, 132, 80, 1028, 40, 50),   # 64-row tiles
    (1, 260, 272, 2052, 25, 333)  # 128-row tiles
])
def test_fp32_products(layers, input_dim, hidden, classes, T, B):
    dims = oracle.ModelDims(layers, input_dim, hidden, classes)
    say(f"fp32 products {layers} {input_dim} {hidden} {classes} N={T * B}")
    master, x, idx, prob, _, _ = _problem(dims, T, B, 3, 0.95, seed=41)
    m = am.Model(layers, input_dim, hidden, classes, am.F32)
    got = gpu_forward_backward(m, master, x, T, B, idx, prob)
    ref = oracle_forward_backward(dims, master, x, T, B, idx, prob)
    _check(got, ref, dims, F32_TOL)
