"""The U draw of Alg. 7 over the whole range of (u, alpha_res, ||Delta_tau||).

One-dimensional blocks put the rejected step's ||Delta|| anywhere from 1e-3 to
300 and alpha_res from 1 down to e^-40, far outside what a sampling run meets,
so that every way the inversion can close is taken: the crossing next to u*
(where the density vanishes), below the first grid, in the far left tail.
The oracle bisects Psi in float64 to the last bit.  Its own rounding moves the
result by about eps / psi(U) relative to the slope of Psi, large only next to
u*: 1e-7 covers it for 24-bit uniforms (1 - u >= 2^-25), and half of all draws
agree to 1e-12.
"""
import numpy as np
import pytest
import torch

from oracle.residual import USAMPLE_EXACT, usample, usample_uniform
from paper_2606_13426_amd import _lib

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("token", [True, False])
@pytest.mark.parametrize("K", [1, 3, 64])
def test_u_draw_over_its_range(token, K):
    B, seed = 1500, 77
    rng = np.random.default_rng(5 + K)
    v = 10.0 ** rng.uniform(-3, 2.5, (B, K))
    z = rng.normal(0, 2.0, (B, K))
    mp = rng.normal(size=(B, K))
    f32 = lambda a: torch.empty(*a.shape, 1, device="cuda").copy_(torch.from_numpy(a)[:, :, None])  # noqa: E731
    mpt = f32(mp)
    mq = torch.cat([f32(mp - v), f32(mp[:, :1])], 1)
    y = f32(mp + z)
    sigma = torch.ones(B, K + 1, dtype=torch.float64, device="cuda")
    kb = torch.full((B,), K, dtype=torch.int32, device="cuda")
    rnd = torch.arange(B, dtype=torch.int32, device="cuda") % 17
    out = _lib.sd_verify_block(y, mpt, mq, sigma, kb, rnd, seed, mode=_lib.SD_TOKEN if token else _lib.SD_BLOCK)
    o = {k: t.cpu().numpy() for k, t in out.items()}
    errs = []
    for b in range(B):
        t = int(o["tau"][b])
        if t > K:
            assert np.isnan(o["u_res"][b])
            continue
        u = usample_uniform(seed, b, b % 17)
        ref = usample(u, float(o["log_alpha_res"][b]), float(o["delta_norm"][b, t - 1]), USAMPLE_EXACT)
        errs.append(abs(o["u_res"][b] - ref) / (1 + abs(ref)))
    assert len(errs) > B // 3
    assert max(errs) <= 1e-7
    assert np.median(errs) <= 1e-12
