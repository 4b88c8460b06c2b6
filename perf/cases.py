"""The calls that programs make of this library, as cases to be timed and checked.

A case is one pass through the public entry points (paper_2606_13426_amd._lib):

  sample  sd_run_sampler_ex: the speculative sampler, a whole run (rounds = 0) or
          its first `rounds` rounds from Y_0 with the state they leave (a run
          served in slices);
  em      sd_run_plain_em: the plain Euler-Maruyama chain;
  target  sd_target_mean: EM means and scores of many rows (a sampling loop of
          the caller's own);
  draft   sd_draft_block;
  verify  sd_verify_block and the residual draw that follows it (a loop with
          the caller's own denoiser between draft and verification).

The shapes are those of the library's own workloads (inputs.WORKLOADS: images
of 3x32x32 and 3x64x64, latents of 4x64x64, a 2-D mixture), of small images
(28x28) and of odd sizes.
"""
import math

import torch

from paper_2606_13426_amd import _lib

DEV = "cuda"
BETA_MIN, BETA_MAX, CHURN = 0.1, 20.0, 1.0
TAG_INIT, TAG_DRAFT, TAG_COIN, TAG_USAMPLE, TAG_RESID, TAG_TARGET = 1, 2, 3, 4, 5, 6


def listed():
    return [
        # the 2-D mixture, whole run: every kernel is tiny, launches and latency count
        dict(name="sample_tiny2d", kind="sample", d=2, M=4, N=100, B=256, K=4, bf16=False, rounds=0,
             token=False, reflect=False, frozen=False),
        # interactive sampling of a few images: 8 chains of 3x32x32, whole run
        dict(name="sample_8x3072", kind="sample", d=3072, M=64, N=200, B=8, K=8, bf16=False, rounds=0,
             token=False, reflect=False, frozen=False),
        # 28x28 images, 100 components (neither a multiple of 64), the paper's
        # baseline variant: token verification with the reflection residual
        dict(name="sample_256x784_token", kind="sample", d=784, M=100, N=250, B=256, K=8, bf16=False, rounds=8,
             token=True, reflect=True, frozen=False),
        # the CIFAR10-sized workload
        dict(name="sample_pixel3072", kind="sample", d=3072, M=64, N=200, B=1024, K=8, bf16=False, rounds=4,
             token=False, reflect=False, frozen=False),
        # 64x64 images, long blocks, bf16 products
        dict(name="sample_pixel12288", kind="sample", d=12288, M=256, N=500, B=512, K=16, bf16=True, rounds=4,
             token=False, reflect=False, frozen=False),
        # the latent-space workload, 1024 components, bf16 products
        dict(name="sample_latent16384", kind="sample", d=16384, M=1024, N=1000, B=256, K=8, bf16=True, rounds=4,
             token=False, reflect=False, frozen=False),
        # the plain chain the sampler is compared with, a batch of 64 images
        dict(name="em_64x3072", kind="em", d=3072, M=64, N=200, B=64, bf16=False),
        # one target call on all rows of a latent-sized round, with scores
        dict(name="target_latent16384", kind="target", d=16384, M=1024, N=1000, rows=2304, bf16=True, score=True),
        # odd sizes throughout: 3x37x37 images, 100 components, rows not aligned
        dict(name="target_odd4107", kind="target", d=4107, M=100, N=200, rows=777, bf16=False, score=True),
        # one draft block of the CIFAR10-sized workload for the caller's denoiser
        dict(name="draft_pixel3072", kind="draft", d=3072, N=200, B=1024, K=8),
        # the largest verification pass: 4096 blocks of 32 drafts of 64x64 images
        dict(name="verify_pixel12288", kind="verify", d=12288, N=1000, B=4096, K=32, token=False, reflect=False),
        # a small verification pass: 64 blocks of 8 drafts, latency counts
        dict(name="verify_64x3072", kind="verify", d=3072, N=250, B=64, K=8, token=False, reflect=False),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _dim(rng, lo, hi):
    """A dimension: any whole number, or a multiple of 4, 64 or 256 as images and latents have."""
    d = _log_uniform(rng, lo, hi)
    q = rng.choice([1, 4, 64, 256])
    return d if d < 2 * q else d // q * q


def draw(rng):
    kind = rng.choice(["sample", "sample", "sample", "sample", "target", "target", "em", "draft", "verify", "verify"])
    if kind == "verify":
        d, K = _dim(rng, 2, 16384), _log_uniform(rng, 1, 32)
        B = _log_uniform(rng, 1, max(1, min(4096, 10 ** 9 // (d * K))))
        token = rng.random() < 0.4
        return dict(kind=kind, d=d, N=rng.choice([100, 250, 500, 1000]), B=B, K=K, token=token,
                    reflect=token and rng.random() < 0.5)
    if kind == "draft":
        d, K = _dim(rng, 2, 16384), _log_uniform(rng, 1, 32)
        B = _log_uniform(rng, 1, max(1, min(4096, 2 * 10 ** 8 // (d * K))))
        return dict(kind=kind, d=d, N=rng.choice([100, 250, 500, 1000]), B=B, K=K)
    d = _dim(rng, 2, 16384)
    M = _dim(rng, 1, 1024)
    bf16 = d >= 1024 and rng.random() < 0.5
    # the work of one pass stays below the largest listed one's
    room = 4 * 10 ** 10 if bf16 else 10 ** 10
    if kind == "target":
        rows = _log_uniform(rng, 1, max(1, min(8192, room // (d * M), 10 ** 8 // d)))
        return dict(kind=kind, d=d, M=M, N=rng.choice([100, 250, 1000]), rows=rows, bf16=bf16,
                    score=rng.random() < 0.5)
    if kind == "em":
        N = rng.choice([50, 100, 200])
        B = _log_uniform(rng, 1, max(1, min(1024, room // (d * M * 10), 10 ** 7 // d)))
        return dict(kind=kind, d=d, M=M, N=N, B=B, bf16=bf16)
    K = _log_uniform(rng, 1, 16)
    B = _log_uniform(rng, 1, max(1, min(1024, room // (d * M * (K + 1)), 10 ** 8 // (d * (K + 1)))))
    token = rng.random() < 0.4
    whole = B * d <= 4096 and B <= 256
    return dict(kind=kind, d=d, M=M, N=100 if whole else rng.choice([250, 500, 1000]), B=B, K=K, bf16=bf16,
                rounds=0 if whole else rng.choice([3, 4, 6]), token=token,
                reflect=token and rng.random() < 0.5, frozen=rng.random() < 0.2)


# ------------------------------------------------------------------ inputs --
def _gen(seed, salt):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 1000003 + salt) & 0x7FFFFFFF)
    return g


def _call_seed(seed):
    return (int(seed) * 2654435761 + 12345) & 0xFFFFFFFFFF


def _mixture(case, seed):
    """mu ~ N(0, I) (N(0, 4I) in a few dimensions), var ~ U[.01, .2], w ~ Dir(1)."""
    g = _gen(seed, 1)
    d, M = case["d"], case["M"]
    mu = torch.randn(M, d, generator=g, device=DEV) * (2.0 if d <= 16 else 1.0)
    var = 0.01 + 0.19 * torch.rand(M, generator=g, device=DEV)
    e = -torch.log(torch.rand(M, generator=g, device=DEV).clamp_min(1e-6))
    return mu, var, torch.log(e / e.sum())


def _signal(N):
    s = 1.0 - torch.arange(N + 1, dtype=torch.float64, device=DEV) / N  # forward time of step n
    return torch.exp(-0.5 * (BETA_MIN * s + 0.5 * (BETA_MAX - BETA_MIN) * s * s))


def _coef(N):
    """(c1, c2, sigma) for n = 0..N in float64."""
    s = 1.0 - torch.arange(N + 1, dtype=torch.float64, device=DEV) / N
    beta = BETA_MIN + s * (BETA_MAX - BETA_MIN)
    return 1.0 + 0.5 * beta / N, 0.5 * (1.0 + CHURN * CHURN) * beta / N, CHURN * torch.sqrt(beta / N)


def _target(case, seed):
    mu, var, log_w = _mixture(case, seed)
    return _lib.Target(_lib.schedule(case["N"], BETA_MIN, BETA_MAX, CHURN), mu.cpu().numpy(), var.cpu().numpy(),
                       log_w.cpu().numpy(), _lib.SD_BF16 if case["bf16"] else _lib.SD_FP32)


def _target_rows(case, seed):
    """Rows as a sampling run meets them: noised mixture draws at steps spread over the schedule."""
    g = _gen(seed, 2)
    mu, var, log_w = _mixture(case, seed)
    rows, d, N = case["rows"], case["d"], case["N"]
    step = torch.randint(0, N, (rows,), generator=g, device=DEV, dtype=torch.int32)
    m = torch.multinomial(log_w.exp(), rows, replacement=True, generator=g)
    a = _signal(N)[step.long()].float()[:, None]
    x0 = mu[m] + var[m].sqrt()[:, None] * torch.randn(rows, d, generator=g, device=DEV)
    x = a * x0 + (1 - a * a).clamp_min(0).sqrt() * torch.randn(rows, d, generator=g, device=DEV)
    return x.contiguous(), step


def _draft_inputs(case, seed):
    g = _gen(seed, 3)
    B, d, N = case["B"], case["d"], case["N"]
    y = torch.randn(B, d, generator=g, device=DEV)
    cache = -y + 0.3 * torch.randn(B, d, generator=g, device=DEV)
    k = torch.randint(0, N, (B,), generator=g, device=DEV, dtype=torch.int32)
    rnd = torch.randint(0, 1 << 16, (B,), generator=g, device=DEV, dtype=torch.int32)
    return y, cache, k, rnd


def _verify_inputs(case, seed):
    """Blocks whose target means lie about half a sigma from the draft means, as where drafts get accepted."""
    g = _gen(seed, 4)
    B, K, d, N = case["B"], case["K"], case["d"], case["N"]
    k0 = torch.randint(0, N, (B,), generator=g, device=DEV)
    left = (N - k0).to(torch.int32)
    kb = torch.minimum(left, torch.full_like(left, K))
    sig = _coef(N)[2]
    sigma = sig[(k0[:, None] + torch.arange(K + 1, device=DEV)).clamp_max(N)].contiguous()
    s32 = sigma.float()[:, :, None]
    mp = torch.randn(B, K, d, generator=g, device=DEV)
    mq = torch.empty(B, K + 1, d, device=DEV)
    mq.normal_(generator=g).mul_(s32 * (0.5 / math.sqrt(d)))
    mq[:, :K] += mp
    mq[:, K] += mp[:, K - 1]
    y = torch.empty(B, K, d, device=DEV)
    y.normal_(generator=g).mul_(s32[:, :K]).add_(mp)
    rnd = torch.randint(0, 1 << 16, (B,), generator=g, device=DEV, dtype=torch.int32)
    return y, mp, mq, sigma, kb, left, rnd


def prepare(case, seed):
    kind, st = case["kind"], dict(case=case, seed=_call_seed(seed))
    if kind in ("sample", "em", "target"):
        st["target"] = _target(case, seed)
    if kind == "sample":
        B, K, d = case["B"], case["K"], case["d"]
        st["ws"] = torch.empty(_lib.sd_sampler_workspace(st["target"], B, K), dtype=torch.uint8, device=DEV)
        st["y"] = torch.zeros(B, d, device=DEV)
        st["trace"] = torch.zeros(case["rounds"] or case["N"], B, dtype=torch.int32, device=DEV)
    elif kind == "em":
        st["ws"] = torch.empty(_lib.sd_plain_em_workspace(st["target"], case["B"]), dtype=torch.uint8, device=DEV)
        st["y"] = torch.empty(case["B"], case["d"], device=DEV)
    elif kind == "target":
        st["x"], st["step"] = _target_rows(case, seed)
        st["mq"] = torch.empty_like(st["x"])
        st["score"] = torch.empty_like(st["x"]) if case["score"] else None
        st["ws"] = torch.empty(_lib.sd_target_mean_workspace(st["target"], case["rows"]), dtype=torch.uint8, device=DEV)
    elif kind == "draft":
        st["y"], st["cache"], st["k"], st["rnd"] = _draft_inputs(case, seed)
        st["sched"] = _lib.schedule(case["N"], BETA_MIN, BETA_MAX, CHURN)
        st["x"] = torch.empty(case["B"], case["K"] + 1, case["d"], device=DEV)
        st["mp"] = torch.empty(case["B"], case["K"], case["d"], device=DEV)
    else:
        st["in"] = _verify_inputs(case, seed)
        B, K = case["B"], case["K"]
        f64 = dict(dtype=torch.float64, device=DEV)
        st["out"] = dict(tau=torch.empty(B, dtype=torch.int32, device=DEV), log_alpha_res=torch.empty(B, **f64),
                         u_res=torch.empty(B, **f64), delta_norm=torch.empty(B, K, **f64),
                         log_ratio=torch.empty(B, K, **f64), coins=torch.empty(B, dtype=torch.int64, device=DEV))
        st["y"] = torch.empty(B, case["d"], device=DEV)
    return st


def run(st):
    c = st["case"]
    kind = c["kind"]
    if kind == "sample":
        y, stats, trace = _lib.sd_run_sampler_ex(
            st["target"], c["B"], c["K"], st["seed"], mode=_lib.SD_TOKEN if c["token"] else _lib.SD_BLOCK,
            residual=_lib.SD_RESIDUAL_REFLECTION if c["reflect"] else _lib.SD_RESIDUAL_DECOMPOSITION,
            drafter=_lib.SD_DRAFTER_FROZEN if c["frozen"] else _lib.SD_DRAFTER_FREE, y_out=st["y"], ws=st["ws"],
            trace=st["trace"], max_rounds=c["rounds"] or -1)
        out = dict(trace=trace, steps=stats["steps"])
        if c["rounds"]:
            v = _lib.sd_sampler_state(st["target"], c["B"], c["K"], st["ws"], stats["rounds"])
            out.update(k=v["k"], mq=v["mq"], cache=v["cache"])
            # with the Frozen Drafter a slice ends before the next block is drafted
            out["x"] = v["x"][:, 0] if c["frozen"] else v["x"]
        else:
            out["y"] = y
        return out
    if kind == "em":
        return _lib.sd_run_plain_em(st["target"], c["B"], st["seed"], y_out=st["y"], ws=st["ws"])
    if kind == "target":
        _lib.sd_target_mean(st["target"], st["x"], st["step"], st["mq"], st["score"], ws=st["ws"])
        return dict(mq=st["mq"], score=st["score"])
    if kind == "draft":
        _lib.sd_draft_block(st["sched"], st["y"], st["cache"], st["k"], st["rnd"], st["seed"], st["x"], st["mp"])
        return dict(x=st["x"], mp=st["mp"])
    y, mp, mq, sigma, kb, left, rnd = st["in"]
    o = _lib.sd_verify_block(y, mp, mq, sigma, kb, rnd, st["seed"],
                             mode=_lib.SD_TOKEN if c["token"] else _lib.SD_BLOCK, out=st["out"])
    if c["reflect"]:
        _lib.sd_sample_residual_reflection(y, mp, mq, sigma, kb, left, o["tau"], rnd, st["seed"], st["y"])
    else:
        _lib.sd_sample_residual(y, mp, mq, sigma, kb, left, o["tau"], o["u_res"], o["delta_norm"], rnd, st["seed"],
                                st["y"])
    return dict(o, y=st["y"])


def work(case):
    """Bytes and operations that a pass cannot do without.  A sampler round needs the target at K + 1 states of each
    chain (two products with the mixture's means), and its drafts and means pass through memory once."""
    kind, d = case["kind"], case["d"]
    if kind == "verify":
        B, K = case["B"], case["K"]
        return dict(bytes=12.0 * B * K * d + 4.0 * B * d, flops=8.0 * B * K * d)
    if kind == "draft":
        B, K = case["B"], case["K"]
        return dict(bytes=4.0 * B * d * (2 + 2 * K + 1), flops=6.0 * B * K * d)
    M, e = case["M"], 2.0 if case["bf16"] else 4.0
    if kind == "target":
        R = case["rows"]
        return dict(bytes=4.0 * R * d * (3 if case["score"] else 2) + e * M * d, flops=4.0 * R * M * d)
    if kind == "em":
        return dict(bytes=case["N"] * (8.0 * case["B"] * d + e * M * d), flops=4.0 * case["N"] * case["B"] * M * d)
    B, K1 = case["B"], case["K"] + 1
    rounds = case["rounds"] or math.ceil(case["N"] / 2)  # a whole run: about two steps a round at these sizes
    if case["frozen"]:
        K1 += 1
    return dict(bytes=rounds * (8.0 * B * K1 * d + e * M * d), flops=4.0 * rounds * B * K1 * M * d)


def tolerance(case):
    """About four times (the whole runs in a few dimensions, which magnify a rounding most) to ten times what the
    library differs by from exact() over many seeds."""
    kind = case["kind"]
    if kind == "verify":
        # float64 sums over float32 rows; y is float32
        return dict(rel=2e-7, max=1e-5)
    if kind == "draft":
        return dict(rel=1e-6, max=1e-4)
    if kind in ("target", "em"):
        # bf16: a softmax weight on a rounding boundary may round the other way
        return dict(rel=2e-4, max=0.1) if case["bf16"] else dict(rel=2e-6, max=1e-4)
    # (a coin within rounding of its threshold may fall the other way in one
    # chain of very many: none did in 200 000 chain-rounds)
    return dict(rel=2e-5, max=1e-3, differ=0.001)


# ------------------------------------------- the same values in 64 bits --
M32 = 0xFFFFFFFF


def _mulhilo(a, b):
    """High and low words of the product of 32-bit words (b a constant)."""
    p, q = (a & 0xFFFF) * b, (a >> 16) * b
    return (q + (p >> 16)) >> 16, (p + ((q & 0xFFFF) << 16)) & M32


def _words(seed, c0, c1, c2, c3):
    """Philox4x32-10 (Salmon et al., SC'11) on int64 tensors holding 32-bit words."""
    k0, k1 = seed & M32, seed >> 32
    c0, c1, c2, c3 = torch.broadcast_tensors(*[torch.as_tensor(v, dtype=torch.int64, device=DEV) for v in (c0, c1, c2, c3)])
    for _ in range(10):
        h0, l0 = _mulhilo(c0, 0xD2511F53)
        h1, l1 = _mulhilo(c2, 0xCD9E8D57)
        c0, c1, c2, c3 = h1 ^ c1 ^ k0, l1, h0 ^ c3 ^ k1, l0
        k0, k1 = (k0 + 0x9E3779B9) & M32, (k1 + 0xBB67AE85) & M32
    return torch.stack([c0, c1, c2, c3], -1)


def _uniform(w):
    return ((w >> 8).double() + 0.5) * 2.0 ** -24


def _normals(seed, chain, rnd, tag, slot, d):
    """[B][d] normals of the chains' streams."""
    w = _words(seed, torch.arange((d + 3) // 4, device=DEV)[None, :], chain[:, None], rnd[:, None], (tag << 24) | slot)
    u = _uniform(w)
    ra, rc = torch.sqrt(-2 * torch.log(u[..., 0])), torch.sqrt(-2 * torch.log(u[..., 2]))
    ta, tc = 2 * math.pi * u[..., 1], 2 * math.pi * u[..., 3]
    z = torch.stack([ra * torch.cos(ta), ra * torch.sin(ta), rc * torch.cos(tc), rc * torch.sin(tc)], -1)
    return z.flatten(1)[:, :d]


class _Exact:
    """m^q and score of the mixture in 64 bits; with bf16 the operands of the two products are rounded first, as
    that precision is defined."""

    def __init__(self, case, seed):
        mu, var, log_w = _mixture(case, seed)
        self.bf16, self.d = case["bf16"], case["d"]
        self.mu, self.var, self.log_w = mu.double(), var.double(), log_w.double()
        self.musq = self.mu.square().sum(1)
        self.mu_op = mu.bfloat16().double() if self.bf16 else self.mu
        self.a = _signal(case["N"])
        self.c1, self.c2, self.sigma = _coef(case["N"])

    def score(self, x, step):
        """Rows x [R][d] in float64, at steps [R]."""
        out = torch.empty_like(x)
        for i in range(0, x.shape[0], 8192):
            xs, n = x[i:i + 8192], step[i:i + 8192].long()
            a = self.a[n][:, None]
            s2 = a * a * self.var[None, :] + (1 - a * a)
            xr = xs.float().bfloat16().double() if self.bf16 else xs
            dist = xs.square().sum(1, keepdim=True) - 2 * a * (xr @ self.mu_op.t()) + a * a * self.musq[None, :]
            r = torch.softmax(self.log_w[None, :] - 0.5 * self.d * torch.log(s2) - dist / (2 * s2), 1)
            rho = (r / s2).sum(1, keepdim=True)
            P = r * a / s2
            P = P.float().bfloat16().double() if self.bf16 else P
            out[i:i + 8192] = P @ self.mu_op - rho * xs
        return out


def _log_excess(x, la, v):
    """log(alpha Phi(x) - Phi(x - v)) for x <= u* = la / v + v / 2: through scaled complementary error functions in
    the left tail, where the two terms nearly cancel."""
    l1 = torch.log(0.5 * torch.special.erfcx(x.abs() / math.sqrt(2)))
    l2 = torch.log(0.5 * torch.special.erfcx((v - x) / math.sqrt(2)))
    lphi = torch.special.log_ndtr(x)
    r = torch.where(x <= 0, (l2 - l1) + v * (x - (la / v + 0.5 * v)), l2 - 0.5 * (x - v) ** 2 - lphi - la)
    return la + lphi + torch.log(-torch.expm1(r.clamp_max(-1e-300)))


def _accept(seed, chain, rnd, ell, vn, kb, token):
    """tau, log alpha_res, U, coins of each chain from ell, ||Delta|| [B][K]."""
    B, K = ell.shape
    j = torch.arange(K, device=DEV)
    w = _words(seed, (j // 4)[None, :], chain[:, None], rnd[:, None], TAG_COIN << 24)
    eta = _uniform(torch.gather(w, 2, (j % 4).expand(B, K)[..., None])[..., 0])
    valid = j[None, :] < kb[:, None]
    la = torch.zeros(B, K, dtype=torch.float64, device=DEV)
    acc = torch.zeros(B, dtype=torch.float64, device=DEV)
    for i in range(K):
        acc = torch.clamp_max(acc + ell[:, i], 0.0)
        la[:, i] = acc
    if token:
        c = valid & (torch.log(eta) < ell.clamp_max(0.0))
        rej = valid & ~c
        tau = torch.where(rej.any(1), rej.int().argmax(1) + 1, kb + 1)
        la_res = torch.zeros(B, dtype=torch.float64, device=DEV)
    else:
        v = torch.cat([vn[:, 1:], torch.ones(B, 1, dtype=torch.float64, device=DEV)], 1)
        vs = torch.where(v > 0, v, torch.ones_like(v))
        lv = _log_excess(la / vs + 0.5 * vs, la, vs)
        lh = lv - torch.logaddexp(lv, torch.log(-torch.expm1(la)))
        lh = torch.where(la >= 0, torch.zeros_like(lh), torch.where(v > 0, lh, torch.full_like(lh, -math.inf)))
        lh = torch.where(j[None, :] + 1 < kb[:, None], lh, la)
        c = valid & (torch.log(eta) < lh)
        tau = torch.where(c, j[None, :] + 2, torch.ones_like(j)[None, :]).amax(1)
        la_res = torch.where(tau >= 2, torch.gather(la, 1, (tau - 2).clamp_min(0)[:, None])[:, 0], torch.zeros_like(acc))
    tau = tau.long()
    coins = (c.long() << j[None, :]).sum(1)
    lu = torch.log(_uniform(_words(seed, torch.zeros_like(chain), chain, rnd, TAG_USAMPLE << 24)[..., 0]))
    v = torch.gather(vn, 1, (tau - 1).clamp(0, K - 1)[:, None])[:, 0]
    draws = (tau <= kb) & (v > 0)
    v = torch.where(draws, v, torch.ones_like(v))
    us = la_res / v + 0.5 * v
    norm = _log_excess(us, la_res, v)
    lo, hi = us - 1.0, us.clone()
    for _ in range(64):
        lo = torch.where(_log_excess(lo, la_res, v) - norm > lu, us - 2 * (us - lo), lo)
    for _ in range(100):
        mid = 0.5 * (lo + hi)
        below = _log_excess(mid, la_res, v) - norm < lu
        lo, hi = torch.where(below, mid, lo), torch.where(below, hi, mid)
    return tau, la_res, torch.where(draws, 0.5 * (lo + hi), torch.full_like(lo, math.nan)), coins


def _rows(t, i):
    return t[torch.arange(t.shape[0], device=DEV), i]


def _residual(seed, chain, rnd, tau, U, kb, left, sigma, y, mp, mq, reflect):
    """The new states; y, mp [B][K][d], mq [B][K+1][d] in float64."""
    K, d = y.shape[1], y.shape[2]
    t = (tau - 1).clamp(0, K - 1)
    q, s = _rows(mq, t), _rows(sigma, t)[:, None]
    D, W = _rows(mp, t) - q, _rows(y, t) - _rows(mp, t)
    nd = D.square().sum(1, keepdim=True)
    if reflect:
        new = _rows(y, t) - (1 + 2 * (D * W).sum(1, keepdim=True) / nd) * D
    else:
        G = _normals(seed, chain, rnd, TAG_RESID, 0, d)
        e = D / nd.sqrt()
        new = q + s * (U[:, None] * e + G - e * (e * G).sum(1, keepdim=True))
    full = _rows(mq, kb) + _rows(sigma, kb)[:, None] * _normals(seed, chain, rnd, TAG_TARGET, 0, d)
    last = _rows(y, (kb - 1).clamp_min(0))
    return torch.where((tau <= kb)[:, None], new, torch.where((kb + 1 <= left)[:, None], full, last))


def _exact_sample(case, seed):
    T, s = _Exact(case, seed), _call_seed(seed)
    B, K, N, d = case["B"], case["K"], case["N"], case["d"]
    chain = torch.arange(B, device=DEV)
    zero = torch.zeros(B, dtype=torch.int64, device=DEV)
    Y, k, r = _normals(s, chain, zero, TAG_INIT, 0, d), zero.clone(), 0
    rows = case["rounds"] or N
    trace = torch.zeros(rows, B, dtype=torch.int32, device=DEV)
    mq_last = torch.zeros(B, K + 1, d, dtype=torch.float64, device=DEV)

    def block(Y, k, r, S):
        x = torch.empty(B, K + 1, d, dtype=torch.float64, device=DEV)
        mp = torch.empty(B, K, d, dtype=torch.float64, device=DEV)
        kb = (N - k).clamp(0, K)
        x[:, 0] = Y
        for i in range(1, K + 1):
            n = (k + i - 1).clamp_max(N)
            m = T.c1[n][:, None] * x[:, i - 1] + T.c2[n][:, None] * S
            z = _normals(s, chain, torch.full_like(k, r), TAG_DRAFT, i, d)
            on = (i <= kb)[:, None]
            mp[:, i - 1] = torch.where(on, m, mp[:, max(i - 2, 0)])
            x[:, i] = torch.where(on, m + T.sigma[n][:, None] * z, x[:, i - 1])
        return x, mp, kb

    S, kc = T.score(Y, k), zero.clone()
    x, mp, kb = block(Y, k, r, S)
    while True:
        on = k < N
        if r >= rows or not bool(on.any()):
            break
        if case["frozen"]:
            x, mp, kb = block(Y, k, r, T.score(Y, k.clamp_max(N - 1)))
        n = (k[:, None] + torch.arange(K + 1, device=DEV)).clamp_max(N - 1)
        score = T.score(x.flatten(0, 1), n.flatten()).view(B, K + 1, d)
        mq = T.c1[n][..., None] * x + T.c2[n][..., None] * score
        sig = T.sigma[(k[:, None] + torch.arange(K + 1, device=DEV)).clamp_max(N)]
        yd = x[:, 1:]
        inv = 1.0 / sig[:, :K]
        D = mp - mq[:, :K]
        vn = D.square().sum(2).sqrt() * inv
        ell = -((yd - mp) * D).sum(2) * inv * inv - 0.5 * vn * vn
        valid = torch.arange(K, device=DEV)[None, :] < kb[:, None]
        ell, vn = torch.where(valid, ell, 0.0), torch.where(valid, vn, 0.0)
        rr = torch.full_like(k, r)
        tau, _, U, _ = _accept(s, chain, rr, ell, vn, kb.clamp_min(1), case["token"])
        new = _residual(s, chain, rr, tau, U, kb, N - k, sig, yd, mp, mq, case["reflect"])
        trace[r] = torch.where(on, tau, 0).int()
        mq_last = torch.where(on[:, None, None], mq, mq_last)
        c = torch.minimum(tau, kb)
        Y = torch.where(on[:, None], new, Y)
        S = torch.where(on[:, None], _rows(score, c), S)
        kc = torch.where(on, (k + c).clamp_max(N - 1), kc)
        k = torch.where(on, (k + tau).clamp_max(N), k)
        r += 1
        if not case["frozen"]:
            x, mp, kb = block(Y, k, r, S)
    out = dict(trace=trace, steps=int(k.sum()))
    if not case["rounds"]:
        return dict(out, y=Y)
    # (after a slice with the Frozen Drafter the library's cache row is the last block's)
    cache = None if case["frozen"] else T.c2[kc][:, None] * S
    return dict(out, k=k.int(), mq=mq_last, cache=cache, x=Y if case["frozen"] else x)


def _exact_verify(case, seed):
    y, mp, mq, sigma, kb, left, rnd = _verify_inputs(case, seed)
    s, K, d = _call_seed(seed), case["K"], case["d"]
    step = max(1, 10 ** 8 // (K * d))
    parts = []
    for i in range(0, case["B"], step):
        c = slice(i, min(case["B"], i + step))
        yc, pc, qc = y[c].double(), mp[c].double(), mq[c].double()
        inv = 1.0 / sigma[c][:, :K]
        D = pc - qc[:, :K]
        vn = D.square().sum(2).sqrt() * inv
        ell = -((yc - pc) * D).sum(2) * inv * inv - 0.5 * vn * vn
        b = kb[c].long()
        valid = torch.arange(K, device=DEV)[None, :] < b[:, None]
        ell, vn = torch.where(valid, ell, 0.0), torch.where(valid, vn, 0.0)
        chain, r = torch.arange(c.start, c.stop, device=DEV), rnd[c].long()
        tau, lar, U, coins = _accept(s, chain, r, ell, vn, b, case["token"])
        new = _residual(s, chain, r, tau, U, b, left[c].long(), sigma[c], yc, pc, qc, case["reflect"])
        parts.append((tau.int(), lar, U, vn, ell, coins, new))
    tau, lar, U, vn, ell, coins, new = (torch.cat(p) for p in zip(*parts))
    return dict(tau=tau, log_alpha_res=lar, u_res=U, delta_norm=vn, log_ratio=ell, coins=coins, y=new)


def exact(case, seed):
    kind = case["kind"]
    if kind == "sample":
        return _exact_sample(case, seed)
    if kind == "verify":
        return _exact_verify(case, seed)
    if kind == "target":
        T = _Exact(case, seed)
        x, step = _target_rows(case, seed)
        x, n = x.double(), step.long()
        sc = T.score(x, n)
        return dict(mq=T.c1[n][:, None] * x + T.c2[n][:, None] * sc, score=sc if case["score"] else None)
    if kind == "em":
        T, s, B, d = _Exact(case, seed), _call_seed(seed), case["B"], case["d"]
        chain = torch.arange(B, device=DEV)
        Y = _normals(s, chain, torch.zeros_like(chain), TAG_INIT, 0, d)
        for n in range(case["N"]):
            nn = torch.full_like(chain, n)
            Y = T.c1[n] * Y + T.c2[n] * T.score(Y, nn) + T.sigma[n] * _normals(s, chain, nn, TAG_TARGET, 1, d)
        return Y
    y, cache, k, rnd = _draft_inputs(case, seed)
    B, K, d, N = case["B"], case["K"], case["d"], case["N"]
    c1, c2, sig = _coef(N)
    x = torch.empty(B, K + 1, d, dtype=torch.float64, device=DEV)
    mp = torch.empty(B, K, d, dtype=torch.float64, device=DEV)
    x[:, 0] = y.double()
    chain, kk = torch.arange(B, device=DEV), k.long()
    for i in range(1, K + 1):
        n = (kk + i - 1).clamp_max(N)
        m = c1[n][:, None] * x[:, i - 1] + c2[n][:, None] * cache.double()
        on = (i <= N - kk)[:, None]
        mp[:, i - 1] = torch.where(on, m, mp[:, max(i - 2, 0)])
        x[:, i] = torch.where(on, m + sig[n][:, None] * _normals(_call_seed(seed), chain, rnd.long(), TAG_DRAFT, i, d),
                              x[:, i - 1])
    return dict(x=x, mp=mp)
