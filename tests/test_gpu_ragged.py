"""Shapes that are no whole number of tiles, chunks or 16-byte rows.

Every float32 target call takes the same matrix-core kernels: partial chunks of
d and M, partial column tiles, a last tile of rows, rows at any 4-byte address.
m^q and the score are compared with float64 on the same float32 inputs.  A
float32 product sum of n terms is off by at most about n 2^-24 of the sum of
magnitudes; with random signs the observed error is near sqrt(n) 2^-24, and
1e-5 of a row's largest value leaves a factor of ten at d = 4100.
"""
import numpy as np
import pytest
import torch

from helpers import assert_rows_close
from oracle import sampler as osamp
from oracle.gmm import GMM
from oracle.schedule import Schedule
from paper_2606_13426_amd import _lib
from paper_2606_13426_amd.inputs import make_gmm

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _reference(p, sched, x, step):
    """m^q and score of rows x at steps, in float64 on the device."""
    tab = torch.from_numpy(_lib.sd_schedule_table(sched)).to(DEV)
    mu, var, lw = (torch.from_numpy(np.asarray(p[k])).to(DEV).double() for k in ("mu", "var", "log_w"))
    a, c1, c2 = (tab[i][step.long()][:, None] for i in (0, 2, 3))
    x = x.double()
    s2 = a * a * var + 1 - a * a
    dist = x.square().sum(1, keepdim=True) - 2 * a * (x @ mu.t()) + a * a * mu.square().sum(1)
    r = torch.softmax(lw - 0.5 * x.shape[1] * torch.log(s2) - dist / (2 * s2), 1)
    sc = (r * a / s2) @ mu - (r / s2).sum(1, keepdim=True) * x
    return c1 * x + c2 * sc, sc


@pytest.mark.parametrize("d,M,rows", [
    (1, 1, 1), (2, 3, 5), (3, 65, 130), (4, 7, 64), (5, 64, 129), (63, 63, 65), (64, 1, 17), (65, 66, 127),
    (127, 100, 128), (130, 129, 3), (784, 100, 300), (1001, 37, 250), (4100, 257, 70),
])
@pytest.mark.parametrize("offset,pad", [(0, 0), (1, 3), (2, 6)])
def test_target_of_any_shape(d, M, rows, offset, pad):
    N = 50
    p = make_gmm(d, M, mu_std=1.0, var=(0.05, 0.4), dirichlet=1.0, seed=d + M)
    sched = _lib.schedule(N)
    tgt = _lib.Target(sched, p["mu"], p["var"], p["log_w"])
    g = torch.Generator(device=DEV)
    g.manual_seed(rows)

    def rows_of(fill):  # rows of stride d + pad that start `offset` floats into an allocation
        t = torch.empty(offset + rows * (d + pad), device=DEV).fill_(fill)
        return t[offset:].view(rows, d + pad)[:, :d]

    # the padding between rows holds NaN: nothing of it may reach a result
    x, mq, sc = rows_of(float("nan")), rows_of(-7.0), rows_of(-7.0)
    x.copy_(torch.randn(rows, d, generator=g, device=DEV))
    step = torch.randint(0, N, (rows,), generator=g, device=DEV, dtype=torch.int32)
    _lib.sd_target_mean(tgt, x, step, mq, sc)
    want_q, want_s = _reference(p, sched, x, step)
    for got, want in ((mq, want_q), (sc, want_s)):
        scale = want.abs().amax(1, keepdim=True)
        assert float(((got.double() - want).abs() / scale).max()) <= 1e-5
    if pad:  # and nothing is written there
        for t in (mq, sc):
            assert bool((t.as_strided((rows - 1, pad), (d + pad, 1), t.storage_offset() + d) == -7.0).all())


@pytest.mark.parametrize("d,M", [(448, 1), (1001, 1), (3, 1), (64, 3), (784, 100)])
def test_single_products_are_rounded_once(d, M):
    # One component far above the others has all the weight, and at x = 0 the score
    # is then P mu, one product an element: float32 arithmetic rounds it once, by
    # 2^-24 at most (5 % more covers the rounding of the split's small terms; the
    # terms that the short form leaves out are 2^-23)
    N, rows = 40, 70
    p = make_gmm(d, M, mu_std=1.0, var=(0.05, 0.4), dirichlet=1.0, seed=d)
    log_w = np.full(M, -2000.0, np.float32)
    log_w[0] = 0.0
    mu = np.array(p["mu"], np.float32)
    mu[1:] = 30.0 * mu[1:]
    sched = _lib.schedule(N)
    tgt = _lib.Target(sched, mu, p["var"], log_w)
    step = torch.arange(rows, device=DEV, dtype=torch.int32) % N
    x = torch.zeros(rows, d, device=DEV)
    mq, sc = torch.empty_like(x), torch.empty_like(x)
    _lib.sd_target_mean(tgt, x, step, mq, sc)
    a = _lib.sd_schedule_table(sched)[0][:N]
    weight = (a * (1.0 / (a * a * float(np.float32(p["var"][0])) + 1.0 - a * a))).astype(np.float32)
    want = torch.from_numpy(weight.astype(np.float64)[step.cpu().numpy(), None] * mu[0].astype(np.float64)).to(DEV)
    assert float(((sc.double() - want).abs() / want.abs()).max()) <= 1.05 * 2.0 ** -24


@pytest.mark.parametrize("d,M,K", [(1, 2, 1), (3, 5, 2), (66, 70, 1), (65, 3, 2), (130, 64, 3), (67, 9, 7)])
def test_sampler_of_any_shape(d, M, K):
    # chains of 2, 3 and 4 rows meet a thread's four rows at every offset
    N, B, seed = 24, 45, 9
    p = make_gmm(d, M, mu_std=1.0, var=(0.05, 0.4), dirichlet=1.0, seed=3)
    tgt = _lib.Target(_lib.schedule(N), p["mu"], p["var"], p["log_w"])
    y, stats, trace = _lib.sd_run_sampler(tgt, B, K, seed, trace_rounds=N)
    torch.cuda.synchronize()
    ref = osamp.run_sampler(GMM(p["mu"], p["var"], p["log_w"]), Schedule(N), B, K, seed)
    y, trace = y.cpu().numpy(), trace.cpu().numpy()
    same = 0
    for i in range(B):
        if any(info["ties"] for info in ref["trace"][i]):
            continue
        taus = [info["tau"] for info in ref["trace"][i]]
        assert list(trace[: len(taus), i]) == taus
        assert_rows_close(y[i][None], ref["y"][i][None], what=f"Y_N chain {i}")
        same += 1
    assert same >= B - 2 and stats["steps"] == B * N


def test_noalloc_rows_in_parts():
    # rows of one component fit the limit, the kernels' padded rows do not: the
    # rows go in parts and give the same bits as one call with a workspace
    d, rows = 3, 420000
    p = make_gmm(d, 1, mu_std=1.0, var=(0.05, 0.4), dirichlet=1.0, seed=1)
    tgt = _lib.Target(_lib.schedule(20), p["mu"], p["var"], p["log_w"])
    assert _lib.sd_target_mean_workspace(tgt, rows) > _lib.sd_target_mean_noalloc_max_bytes()
    x = torch.randn(rows, d, device=DEV)
    step = torch.randint(0, 20, (rows,), device=DEV, dtype=torch.int32)
    a, b, sa, sb = (torch.empty_like(x) for _ in range(4))
    _lib.sd_target_mean(tgt, x, step, a, sa)
    _lib.sd_target_mean_noalloc(tgt, x, step, b, sb)
    assert torch.equal(a, b) and torch.equal(sa, sb)
