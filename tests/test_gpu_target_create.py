"""What a target holds on the device, and means that reach it in several slices."""
import numpy as np
import pytest
import torch

from paper_2606_13426_amd import _lib
from paper_2606_13426_amd.inputs import make_gmm

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("bf16", [False, True])
def test_target_holds_its_operand_planes_only(bf16):
    # three planes (bf16: one) of mu and of mu^T, the tables (no smaller than one
    # 8 MB slice of mu) and the allocator's rounding; no float32 copy of mu (64 MB)
    d, M = 16384, 1024
    p = make_gmm(d, M, mu_std=1.0, var=(0.05, 0.4), dirichlet=1.0, seed=1)
    make = lambda: _lib.Target(_lib.schedule(20), p["mu"], p["var"], p["log_w"],  # noqa: E731
                               _lib.SD_BF16 if bf16 else _lib.SD_FP32)
    make()  # (a device's first use takes memory of its own)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    tgt = make()
    held = free - torch.cuda.mem_get_info()[0]
    planes = (1 if bf16 else 3) * 2 * 2 * M * d
    assert tgt.d == d and planes <= held <= planes + (16 << 20)


# 8 MB of mu at a time in blocks of 32 components: one slice, several with a last one
# of 32, of 8 and of 5 components, and the least of 32 (rows of 400 KB)
@pytest.mark.parametrize("d,M", [(2048, 1024), (32769, 64), (16388, 1000), (4099, 485), (100003, 70)])
@pytest.mark.parametrize("bf16", [False, True])
def test_every_slice_of_the_means_arrives(d, M, bf16):
    # row m lies at component m's mean, far from every other: its score is
    # P_m mu_m - x / s2, each term off by a float32 rounding or two of its size
    N = 10
    p = make_gmm(d, M, mu_std=1.0, var=(0.2, 0.2), dirichlet=1.0, seed=2)
    mu = np.array(p["mu"], np.float32)
    sched = _lib.schedule(N)
    tgt = _lib.Target(sched, mu, p["var"], np.zeros(M, np.float32), _lib.SD_BF16 if bf16 else _lib.SD_FP32)
    a, _, _, _ = _lib.sd_schedule_table(sched)[:, N - 1]
    mt = torch.from_numpy(mu).to(DEV)
    x = (float(a) * mt).contiguous()
    mq, sc = torch.empty_like(x), torch.empty_like(x)
    _lib.sd_target_mean(tgt, x, torch.full((M,), N - 1, dtype=torch.int32, device=DEV), mq, sc)
    s2 = a * a * np.float64(p["var"][0]) + 1 - a * a
    rnd = (lambda t: t.bfloat16().double()) if bf16 else (lambda t: t.double())
    weight = rnd(torch.tensor(a / s2, device=DEV).float())
    want = weight * rnd(mt) - x.double() / s2
    assert float((sc.double() - want).abs().max()) <= 2.0 ** -21 * float((x.abs() / s2).max())
