"""GPU parity of target generation at the sizes where its kernels change
course: the k-best selection with one and two groups a lane, rows that are
nearly all candidates, ties that overflow them; posteriors of partial tiles
and of rows longer than a tile; the valid-row count of unaligned masks."""

import numpy as np
import pytest
import torch

import oracle
from paper_1904_10584_amd import binding as am
from tests.gpu_util import say, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C,K", [(4, 4), (33, 33), (64, 32), (100, 53), (128, 64), (129, 64), (256, 33),
                                 (412, 53), (1000, 32), (1024, 33), (2050, 64), (4096, 1), (8192, 64)])
def test_kbest_logits_bounds(C, K):
    rng = np.random.default_rng(C * 65 + K)
    N = 203
    z = (rng.standard_normal((N, C)) * 3).astype(np.float32)
    z[1] = 1.5                                   # all equal: every entry is a candidate
    z[2, : C // 2] = 7.0                         # half of the row at the maximum
    z[3] = np.sort(z[3])                         # neighbours in one lane's registers
    z[4] = np.sort(z[4])[::-1]
    z[5] = np.nan
    z[6, rng.integers(0, C, C // 2 + 1)] = np.nan
    z[7] = -np.inf
    z[8, 0] = np.inf
    z[9] = np.round(z[9])
    z[10, ::2] = np.float32(-3.4028235e38)
    z[11] = 0.0
    z[11, ::3] = -0.0
    say(f"kbest C={C} K={K}")
    idx = torch.empty((N, K), dtype=torch.int32, device="cuda")
    val = torch.empty((N, K), dtype=torch.float32, device="cuda")
    am.kbest_logits(to_dev(z), idx, val)
    ri, rv = oracle.topk_logits(z, K)
    np.testing.assert_array_equal(idx.cpu().numpy(), ri)
    np.testing.assert_array_equal(val.cpu().numpy().view(np.uint32), rv.astype(np.float32).view(np.uint32))


# both sides of the lines where few k of short rows are left to rounds, and short
# rows that nearly all reach the bound; more than 128 equal values at the bound with any
# number above it, whole and partial blocks of registers, aligned rows or not
@pytest.mark.parametrize("C,K", [(64, 1), (256, 4), (256, 5), (257, 8), (512, 9), (513, 9), (768, 10), (769, 10),
                                 (1024, 11), (1025, 7), (2048, 8), (2049, 1), (200, 50), (256, 64), (640, 20), (641, 20), (3000, 20), (3001, 20), (5000, 33),
                                 (6147, 64), (8192, 32)])
def test_kbest_logits_routes_and_ties(C, K):
    rng = np.random.default_rng(C * 67 + K)
    N = 131
    z = rng.standard_normal((N, C)).astype(np.float32)
    for r in range(N - 40):  # equal values, r % (K + 40) larger ones, the rest below
        above = r % (K + 40)
        z[r] = np.float32(-r)
        z[r, rng.permutation(C)[:C // 5]] -= 1.0
        at = rng.permutation(C)[:above]
        z[r, at] = rng.integers(1, 5, len(at)) if r % 2 else rng.uniform(1, 5, len(at))
        if r % 3 == 0:
            z[r, rng.permutation(C)[:C // 7]] = np.nan
        if r % 7 == 0:
            z[r] = np.where(z[r] == -r, np.float32(np.nan), z[r])
    z[-1] = -np.inf
    z[-2] = np.where(np.arange(C) % 2 == 1, np.float32(0.0), np.float32(-0.0))
    say(f"kbest routes C={C} K={K}")
    idx = torch.empty((N, K), dtype=torch.int32, device="cuda")
    val = torch.empty((N, K), dtype=torch.float32, device="cuda")
    am.kbest_logits(to_dev(z), idx, val)
    ri, rv = oracle.topk_logits(z, K)
    np.testing.assert_array_equal(idx.cpu().numpy(), ri)
    np.testing.assert_array_equal(val.cpu().numpy().view(np.uint32), rv.astype(np.float32).view(np.uint32))


@pytest.mark.parametrize("N,K", [(1, 1), (63, 20), (130, 64), (67, 65), (5, 1000), (3, 4096), (3, 4097)])
def test_kbest_posterior_tiles(N, K):
    rng = np.random.default_rng(N + K)
    v = np.sort(rng.standard_normal((N, K)) * 4, axis=1)[:, ::-1].astype(np.float32)
    v[0, -1] = -np.inf
    say(f"posteriors N={N} K={K}")
    prob = torch.empty((N, K), dtype=torch.float32, device="cuda")
    am.kbest_posteriors(to_dev(v.copy()), prob)
    got = prob.cpu().numpy()
    if K == 1:
        return np.testing.assert_array_equal(np.isnan(got), True)  # -inf - -inf, as before
    # one fp32 sum of K terms in order: K half-ulps
    np.testing.assert_allclose(got, oracle.kbest_posteriors(v), rtol=max(2e-6, K * 6e-8), atol=1e-30)


@pytest.mark.parametrize("N,offset", [(1, 0), (7, 3), (15, 1), (33, 15), (4099, 5), (70001, 0)])
def test_mean_over_masked_rows(N, offset):
    # logits all zero, one class with probability 1: each valid row's loss is
    # log C, so the mean is log C whatever rows are masked
    C = 8
    rng = np.random.default_rng(N)
    bits = (rng.random(N) < 0.4).astype(np.uint8) * rng.integers(1, 256, N).astype(np.uint8)
    bits[-1] = 128
    say(f"mask N={N} offset={offset}")
    whole = torch.zeros(N + 16, dtype=torch.uint8, device="cuda")
    mask = whole[offset:offset + N]
    mask.copy_(torch.from_numpy(bits))
    z = torch.zeros((N, C), device="cuda")
    idx = torch.zeros((N, 1), dtype=torch.int32, device="cuda")
    prob = torch.ones((N, 1), device="cuda")
    loss = torch.zeros(1, device="cuda")
    dz = torch.full((N, C), 9.0, device="cuda")
    ws = torch.zeros(am.ce_workspace_bytes(N), dtype=torch.uint8, device="cuda")
    am.sparse_soft_ce(z, idx, prob, loss, dz, ws, mask=mask)
    valid = int((bits != 0).sum())
    # each row's 1 / valid and the tree sum are rounded: far under 1e-5
    assert abs(float(loss[0]) - np.log(C)) < 1e-5
    got = dz.cpu().numpy()
    np.testing.assert_array_equal(got[bits == 0], 0.0)
    np.testing.assert_allclose(got[bits != 0][:, 1], 1.0 / C / valid, rtol=1e-6)
