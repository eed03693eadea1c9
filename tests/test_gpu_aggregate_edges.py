"""GPU parity of the decoders at the sizes where they change course: more
streams than one table of ranges holds, tiles with many words of a stream,
streams without words, unaligned outputs, lengths that are no
multiple of four."""

import numpy as np
import pytest
import torch

import oracle
from paper_1904_10584_amd import binding as am
from tests.gpu_util import say, to_dev

pytestmark = pytest.mark.gpu


def _streams(n, S, rate, rng):
    rows = []
    for s in range(S):
        at = np.flatnonzero(rng.random(n) < (0.0 if s % 7 == 3 else rate))
        rows.append(((at.astype(np.uint32) << 1) | rng.integers(0, 2, at.size).astype(np.uint32)))
    cap = max(1, max(r.size for r in rows))
    words = np.full((S, cap), 0xFFFFFFFF, np.uint32)
    for s, r in enumerate(rows):
        words[s, :r.size] = r
    return words, np.array([r.size for r in rows], np.int64)


def _offset_dense(base, off):
    whole = torch.full((base.size + 8,), 5.0, device="cuda")
    d = whole[off:off + base.size]
    d.copy_(torch.from_numpy(base))
    return whole, d


@pytest.mark.parametrize("n,S,rate", [(3, 2, 0.9), (4095, 16, 0.5), (12289, 65, 0.05), (8192, 130, 1.0),
                                      (40_003, 17, 0.003),
                                      # waves' shares that differ: by the whole workgroup
                                      # where a range is long, else by the waves
                                      (12_289, 1, 0.9), (8192, 1, 0.015), (8192, 2, 0.3), (4096, 3, 0.015),
                                      (20_000, 5, 0.5), (20_000, 6, 0.1), (9001, 67, 0.4), (9001, 69, 0.1)])
@pytest.mark.parametrize("accumulate", [False, True])
@pytest.mark.parametrize("off", [0, 1])
def test_decode_multi_edges(n, S, rate, accumulate, off):
    rng = np.random.default_rng(n + S)
    words, counts = _streams(n, S, rate, rng)
    tau = np.float32(1e-4)
    base = rng.standard_normal(n).astype(np.float32)
    base[::5] = -0.0
    say(f"decode_multi edges n={n} S={S} rate={rate} acc={accumulate} off={off}")
    whole, dense = _offset_dense(base, off)
    ws = torch.zeros(max(256, am.decode_multi_workspace_bytes(S, n)), dtype=torch.uint8, device="cuda")
    am.grad_threshold_decode_multi(to_dev(words.view(np.int32)), to_dev(counts), tau, dense, ws,
                                   accumulate=accumulate)
    ref = oracle.grad_threshold_decode_multi(words, counts, tau, n, base, accumulate)
    np.testing.assert_array_equal(dense.cpu().numpy().view(np.uint32), ref.astype(np.float32).view(np.uint32))
    outside = torch.cat([whole[:off], whole[off + n:]])
    assert bool((outside == 5.0).all())


@pytest.mark.parametrize("n", [1, 4095, 4098, 50_001])
@pytest.mark.parametrize("accumulate", [False, True])
@pytest.mark.parametrize("off", [0, 2])
def test_decode_edges(n, accumulate, off):
    rng = np.random.default_rng(n)
    words, counts = _streams(n, 1, 0.3, rng)
    tau = np.float32(1e-3)
    base = rng.standard_normal(n).astype(np.float32)
    say(f"decode edges n={n} acc={accumulate} off={off}")
    whole, dense = _offset_dense(base, off)
    am.grad_threshold_decode(to_dev(words[0].view(np.int32)), to_dev(counts), tau, dense, accumulate)
    ref = oracle.grad_threshold_decode(words[0], int(counts[0]), tau, n, base, accumulate)
    np.testing.assert_array_equal(dense.cpu().numpy().view(np.uint32), ref.astype(np.float32).view(np.uint32))
    outside = torch.cat([whole[:off], whole[off + n:]])
    assert bool((outside == 5.0).all())
