"""The target time that bench.py forms its speedup terms from."""
import pytest
import torch

import bench
from paper_2606_13426_amd import _lib
from paper_2606_13426_amd.inputs import make_gmm


def test_target_time_counts_every_kernel_of_a_target_call():
    prof = {"init_chains": (1, 1.0), "gmm_logits": (3, 2.0), "gmm_softmax": (3, 4.0), "em_step": (3, 8.0),
            "scan_fused": (3, 16.0), "em_step_bf16_big": (1, 32.0)}
    assert bench.target_us(prof) == 1e3 * (2.0 + 4.0 + 8.0 + 32.0)


@pytest.mark.gpu
@pytest.mark.parametrize("d,M,B,bf16", [(64, 8, 5, False), (1024, 64, 33, True), (16384, 512, 864, True)])
def test_a_plain_chain_is_its_target_calls(d, M, B, bf16):
    # three kernels a step and the chains' start: all but the start are the target's
    N = 3
    p = make_gmm(d, M, mu_std=1.0, var=(0.05, 0.4), dirichlet=1.0, seed=1)
    tgt = _lib.Target(_lib.schedule(N), p["mu"], p["var"], p["log_w"], _lib.SD_BF16 if bf16 else _lib.SD_FP32)
    _lib.sd_profile_enable(True)
    _lib.sd_run_plain_em(tgt, B, 7)
    torch.cuda.synchronize()
    prof = _lib.sd_profile_read()
    _lib.sd_profile_enable(False)
    start = prof.pop("init_chains")
    assert start[0] == 1 and sum(n for n, _ in prof.values()) == 3 * N
    assert bench.target_us(prof) == pytest.approx(1e3 * sum(ms for _, ms in prof.values()))
