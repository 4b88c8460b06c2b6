"""The target's softmax at logits far from zero.

A row far from the data at a late step has logits of -||x||^2 / (2 s^2): 1e10 and
more, where a maximum rounded to float32 is off by more than the exponential's
range.  m^q and the score stay finite and equal to float64 on the same operands
(bf16: rounded as that precision defines).  The products' float32 sums bound the
error: 1e-5 of a row's largest value, as in test_gpu_ragged.py, and with bf16 the
weights beside a rounding boundary: 2^-8 of P mu, whose size is a few means' entries
against x's in the row's largest value.
"""
import numpy as np
import pytest
import torch

from paper_2606_13426_amd import _lib
from paper_2606_13426_amd.inputs import make_gmm

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _reference(p, sched, x, step, bf16):
    """m^q and score of rows x at one step, in float64 on the device."""
    a, _, c1, c2 = (float(t[step]) for t in _lib.sd_schedule_table(sched))
    mu, var, lw = (torch.from_numpy(np.asarray(p[k])).to(DEV).double() for k in ("mu", "var", "log_w"))
    rnd = (lambda t: t.bfloat16().double()) if bf16 else (lambda t: t.double())
    mo, xd = rnd(mu.float()), x.double()
    s2 = a * a * var + 1 - a * a
    dist = xd.square().sum(1, keepdim=True) - 2 * a * (rnd(x) @ mo.t()) + a * a * mu.square().sum(1)
    r = torch.softmax(lw - 0.5 * x.shape[1] * torch.log(s2) - dist / (2 * s2), 1)
    sc = rnd((r * a / s2).float()) @ mo - (r / s2).sum(1, keepdim=True) * xd
    return c1 * xd + c2 * sc, sc


# every way a row is held: one to sixteen wavefronts of one component a lane, and
# (from 4096 wavefronts on, 10240 of up to 64 components) a quarter and a half of a
# wavefront, one, two and four of four components; last workgroups that are not full
@pytest.mark.parametrize("M,rows", [(5, 70), (100, 33), (200, 40), (400, 40), (1000, 40), (5, 10245), (64, 10240), (65, 2050),
                                    (100, 2049), (130, 1367), (300, 831), (600, 427)])
@pytest.mark.parametrize("scale", [3.0, 5e3, 6e4, 1e20])
@pytest.mark.parametrize("bf16", [False, True])
def test_logits_far_from_zero(M, rows, scale, bf16):
    if bf16 and scale > 1e18:
        scale = 1e15  # (||x||^2 of bf16 targets may be summed from float32 squares)
    d, N = 64, 50
    p = make_gmm(d, M, mu_std=1.0, var=(0.05, 0.4), dirichlet=1.0, seed=M)
    sched = _lib.schedule(N)
    tgt = _lib.Target(sched, p["mu"], p["var"], p["log_w"], _lib.SD_BF16 if bf16 else _lib.SD_FP32)
    g = torch.Generator(device=DEV)
    g.manual_seed(rows)
    x = scale * torch.randn(rows, d, generator=g, device=DEV)
    mq, sc = torch.empty_like(x), torch.empty_like(x)
    _lib.sd_target_mean(tgt, x, torch.full((rows,), N - 1, dtype=torch.int32, device=DEV), mq, sc)
    tol = 1e-5 + (2.0 ** -7 / scale if bf16 else 0.0)
    for got, want in zip((mq, sc), _reference(p, sched, x, N - 1, bf16)):
        assert bool(torch.isfinite(got).all())
        assert float(((got.double() - want).abs() / want.abs().amax(1, keepdim=True)).max()) <= tol
