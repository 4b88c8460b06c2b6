"""Both sides of the rules that pick a kernel by size.

Draft blocks of few chains are spread over the wavefronts of a workgroup, the
float32 logits split d over up to 64 workgroups, a bf16 public call of many rows
runs on 288 x 256 tiles and a plain Euler-Maruyama step adds its noise in the
target call's last kernel.  Each is compared with the path it stands in for:
bit for bit where the arithmetic is the same, else with float64 (float32 sums:
1e-5 of a row's largest value, as in test_gpu_ragged.py) or, for the same bf16
operands summed in another order, to 2^-19 of a row's largest value (sums of
1024 float32 terms are off by about sqrt(1024) 2^-24 of their size).
"""
import numpy as np
import pytest
import torch

from paper_2606_13426_amd import _lib
from paper_2606_13426_amd.inputs import make_gmm
from test_gpu_ragged import _reference

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _draft(B, K, d, y, cs, k, rnd, off, pad):
    """The draft block of the first B chains, rows of stride d + pad, `off` floats into an allocation."""
    def block(rows):
        t = torch.full((off + B * rows * (d + pad),), 7.0, device=DEV)
        return t[off:].view(B, rows, d + pad)[:, :, :d]

    x, mp = block(K + 1), block(K)
    _lib.sd_draft_block(_lib.schedule(90), y[:B].contiguous(), cs[:B].contiguous(), k[:B].contiguous(),
                        rnd[:B].contiguous(), 77, x, mp)
    return x, mp


@pytest.mark.parametrize("K,d", [(2, 1), (3, 63), (4, 256), (5, 257), (15, 130), (16, 256), (17, 255), (33, 64), (64, 9)])
@pytest.mark.parametrize("off,pad", [(0, 0), (1, 0), (0, 3), (4, 4)])
def test_spread_draft_equals_one_thread_per_group(K, d, off, pad):
    # at most 1024 wavefronts' worth of groups are spread, more are not
    big = 1024 // ((d + 255) // 256) + 1
    g = torch.Generator(device=DEV)
    g.manual_seed(K)
    y, cs = (torch.randn(big, d, generator=g, device=DEV) for _ in range(2))
    k = torch.randint(0, 92, (big,), generator=g, device=DEV, dtype=torch.int32)  # some chains are done
    k[0], k[1], k[2] = 0, 89, 90 - min(K, 5)
    rnd = torch.randint(0, 99, (big,), generator=g, device=DEV, dtype=torch.int32)
    want = _draft(big, K, d, y, cs, k, rnd, off, pad)
    for B in (1, 3, big - 1):
        for a, b in zip(_draft(B, K, d, y, cs, k, rnd, off, pad), want):
            assert torch.equal(a, b[:B])


# blocks of one row take a kernel of their own: the first row of blocks of two, whose
# chains here are too many to be spread
@pytest.mark.parametrize("d", [1, 4, 63, 256, 1030])
@pytest.mark.parametrize("off,pad", [(0, 0), (1, 3), (4, 4)])
def test_single_draft_is_the_first_of_two(d, off, pad):
    B = 1024 // ((d + 255) // 256) + 1
    g = torch.Generator(device=DEV)
    g.manual_seed(d)
    y, cs = (torch.randn(B, d, generator=g, device=DEV) for _ in range(2))
    k = torch.randint(0, 92, (B,), generator=g, device=DEV, dtype=torch.int32)  # some chains are done
    rnd = torch.randint(0, 99, (B,), generator=g, device=DEV, dtype=torch.int32)
    x1, m1 = _draft(B, 1, d, y, cs, k, rnd, off, pad)
    x2, m2 = _draft(B, 2, d, y, cs, k, rnd, off, pad)
    assert torch.equal(x1, x2[:, :2]) and torch.equal(m1, m2[:, :1])


# 33 to 64 chunks of d on one tile of rows: a workgroup each; 65: two each
@pytest.mark.parametrize("d,M,rows", [(2112, 64, 72), (3072, 64, 1), (4096, 70, 128), (4095, 64, 100), (4160, 64, 72), (4161, 3, 20),
                                      # rows that share a wavefront, 6 and 15 splits
                                      (3072, 64, 10243), (9000, 100, 2050)])
def test_logits_over_many_splits(d, M, rows):
    N = 50
    p = make_gmm(d, M, mu_std=1.0, var=(0.05, 0.4), dirichlet=1.0, seed=d)
    sched = _lib.schedule(N)
    tgt = _lib.Target(sched, p["mu"], p["var"], p["log_w"])
    g = torch.Generator(device=DEV)
    g.manual_seed(rows)
    # rows between two components, so that the logits' errors reach the weights
    mu = torch.from_numpy(np.asarray(p["mu"])).to(DEV).float()
    x = (0.5 * (mu[torch.arange(rows, device=DEV) % M] + mu[torch.arange(rows, device=DEV) * 7 % M])
         + 0.3 * torch.randn(rows, d, generator=g, device=DEV)).contiguous()
    step = torch.randint(0, N // 2, (rows,), generator=g, device=DEV, dtype=torch.int32)
    mq = torch.empty_like(x)
    _lib.sd_target_mean(tgt, x, step, mq)
    want, _ = _reference(p, sched, x, step)
    assert float(((mq.double() - want).abs() / want.abs().amax(1, keepdim=True)).max()) <= 1e-5


def _bf16_target(d, M, N):
    # components that overlap: a row's weights spread over many of them (apart, one
    # has all the weight and the order of the sums could not show)
    p = make_gmm(d, M, mu_std=0.01, var=(0.2, 0.2), dirichlet=1.0, seed=M)
    return _lib.Target(_lib.schedule(N), p["mu"], p["var"], p["log_w"], _lib.SD_BF16)


def _launches(call, *names):
    """The launches of the kernels `names` during call(), and its result."""
    _lib.sd_profile_enable(True)
    out = call()
    n = [_lib.sd_profile_seen(k) for k in names]
    _lib.sd_profile_enable(False)
    return n, out


# 864 = 3 tiles of 288 rows (192 of 256 workgroups: the least that takes them),
# 1100 and 1151: a last tile of 236 and 287 rows
@pytest.mark.parametrize("d,M,rows", [(16384, 512, 864), (16384, 576, 1100), (16384, 512, 1151), (16640, 1024, 863)])
@pytest.mark.parametrize("pad", [0, 4])
def test_public_mean_tiles_agree(d, M, rows, pad):
    N = 60
    tgt = _bf16_target(d, M, N)
    g = torch.Generator(device=DEV)
    g.manual_seed(rows)
    x = torch.full((rows, d + pad), float("nan"), device=DEV)[:, :d]
    x.copy_(torch.randn(rows, d, generator=g, device=DEV))
    step = torch.randint(0, N, (rows,), generator=g, device=DEV, dtype=torch.int32)

    def call(extra, score):  # rows of stride d + extra: 16-byte aligned where extra % 4 == 0
        mq, sc = (torch.full((rows, d + extra), -7.0, device=DEV) for _ in range(2))
        _lib.sd_target_mean(tgt, x, step, mq[:, :d], sc[:, :d] if score else None)
        assert extra == 0 or bool((mq[:, d:] == -7.0).all()) and bool((sc[:, d:] == -7.0).all())
        return mq[:, :d], sc[:, :d]

    kernels = ("gmm_mean_bf16_big", "gmm_mean_bf16")
    n, big = _launches(lambda: call(pad, True), *kernels)
    assert n == [1, 0]
    n, small = _launches(lambda: call(1, True), *kernels)
    assert n == [0, 1]
    for a, b in zip(big, small):
        assert float(((a - b).abs() / b.abs().amax(1, keepdim=True)).max()) <= 2.0 ** -19
    assert torch.equal(call(pad, False)[0], big[0])


def test_public_mean_tiles_begin_at_three_quarters_of_a_wave():
    tgt = _bf16_target(16384, 512, 10)
    for rows, want in ((863, [0, 1]), (864, [1, 0])):
        x = torch.zeros(rows, 16384, device=DEV)
        step = torch.zeros(rows, dtype=torch.int32, device=DEV)
        n, _ = _launches(lambda: _lib.sd_target_mean(tgt, x, step, torch.empty_like(x)), "gmm_mean_bf16_big", "gmm_mean_bf16")
        assert n == want, rows


# (3, 1) the float32 kernels, bf16 on 128 x 128 tiles, and on 288 x 256 ones
@pytest.mark.parametrize("d,M,B,bf16", [(3, 5, 70, False), (66, 64, 65, False), (128, 100, 5, False), (256, 64, 64, False),
                                        (1024, 96, 130, True), (1028, 64, 33, True), (16384, 512, 864, True)])
@pytest.mark.parametrize("N", [1, 2, 3])
def test_plain_step_is_mean_plus_noise(d, M, B, bf16, N):
    p = make_gmm(d, M, mu_std=1.0, var=(0.05, 0.4), dirichlet=1.0, seed=d)
    sched = _lib.schedule(N)
    tgt = _lib.Target(sched, p["mu"], p["var"], p["log_w"], _lib.SD_BF16 if bf16 else _lib.SD_FP32)
    seed = 41
    # (an odd and an even number of steps end in y_out from either buffer)
    got = _lib.sd_run_plain_em(tgt, B, seed, y_out=torch.full((B, d), 9.0, device=DEV))
    y = torch.empty(B, d, device=DEV)
    _lib.sd_init_chains(y, seed)
    sigma = _lib.sd_schedule_table(sched)[1]
    for n in range(N):
        mq, z = torch.empty_like(y), torch.empty_like(y)
        _lib.sd_target_mean(tgt, y, torch.full((B,), n, dtype=torch.int32, device=DEV), mq)
        for b in range(B):
            _lib.sd_philox_normals(seed, b, n, 6, 1, z[b])
        # the kernel rounds the sum once (a fused multiply-add), as float64 does here
        y = (mq.double() + float(np.float32(sigma[n])) * z.double()).float()
    assert float((got - y).abs().max()) <= 2.0 ** -19 * float(y.abs().max())


def _state(tgt, B, K, rounds, groups):
    """A slice's statistics, trace and the state it leaves; its workspace, to go on from."""
    ws = torch.zeros(_lib.sd_sampler_workspace(tgt, B, K), dtype=torch.uint8, device=DEV)
    trace = torch.zeros(40, B, dtype=torch.int32, device=DEV)
    _, st, _ = _lib.sd_run_sampler_ex(tgt, B, K, 0, max_rounds=rounds, groups=groups, ws=ws, trace=trace)
    v = _lib.sd_sampler_state(tgt, B, K, ws, st["rounds"])
    keep = ("x", "k", "round", "cache", "cache_step", "mq", "lrp", "tau", "coins", "log_alpha_res", "ties")
    return st, trace, {k: v[k].clone() for k in keep}, ws


def test_slices_choose_one_group():
    # the choice by rows holds for calls that run many rounds; a slice of few
    # takes one group, with the same state as any grouping
    p = make_gmm(64, 8, mu_std=1.0, var=(0.01, 0.2), dirichlet=1.0, seed=1)
    tgt = _lib.Target(_lib.schedule(40), p["mu"], p["var"], p["log_w"])
    B, K = 456, 8
    y, whole, trace = _lib.sd_run_sampler_ex(tgt, B, K, 0, trace_rounds=40)
    assert whole["groups"] == 2 and whole["finished"]
    for rounds, want in ((4, 1), (7, 1), (8, 2), (32, 2)):
        st, tr, state, ws = _state(tgt, B, K, rounds, 0)
        assert st["groups"] == want, (rounds, st["groups"])
        for groups in (1, 2):
            st2, tr2, state2, _ = _state(tgt, B, K, rounds, groups)
            assert st2["groups"] == groups and torch.equal(tr, tr2)
            for k in state:
                assert torch.equal(state[k], state2[k]), (rounds, groups, k)
        # the run continued from the slice equals the whole call
        y2, st, _ = _lib.sd_run_sampler_ex(tgt, B, K, 0, start_round=st["rounds"], ws=ws, trace=tr)
        assert torch.equal(y, y2) and torch.equal(trace, tr)
        assert all(st[k] == whole[k] for k in ("rounds", "steps", "ties", "tau_hist"))


# 456 blocks of 9 rows: the largest d within 256 MB, and one more
@pytest.mark.parametrize("d,want", [(16352, 1), (16353, 2)])
def test_slices_of_blocks_past_the_infinity_cache_keep_two_groups(d, want):
    p = make_gmm(d, 3, mu_std=1.0, var=(0.01, 0.2), dirichlet=1.0, seed=1)
    tgt = _lib.Target(_lib.schedule(40), p["mu"], p["var"], p["log_w"])
    st, tr, state, ws = _state(tgt, 456, 8, 2, 0)
    assert st["groups"] == want and (456 * 9 * 4 * d > 256 << 20) == (want == 2)
    del ws
    _, tr2, state2, ws = _state(tgt, 456, 8, 2, 3 - want)
    assert torch.equal(tr, tr2) and all(torch.equal(state[k], state2[k]) for k in state)
