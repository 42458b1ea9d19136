"""Work that users of the sampler have it do, from the smallest calls to plateau-sized ones.

Every case is one call of the public binding (``Sampler.sample``,
``Sampler.sample_batch`` or ``Sampler.sample_stored``) on a chain made from
the seed, returning what the call returns: the outcomes of every sample at
every site and the samples' log-probabilities.

A case is a dict of plain values:

  call       "sample", "batch" or "stored"
  precision  the handle's form (fp32, fp16f6, fp16f8, bf16x3, fp16x3)
  M          sites (batch: the shortest chain's)
  M_hi       batch: the longest chain's sites
  d, d_hi    physical dimension; d_k is uniform on {d .. d_hi}
  chi        bond cap (the bonds ramp up from the open ends as far as
             products of d_k allow); batch: the largest cap of the ensemble
  N          samples of the call (batch: of every chain)
  B          batch: chains
  sigma      scale of the per-sample displacements (0: none)
  storage    stored: "cf16" or "cf8"
  host       stored: the sites are in pinned host memory (else on the GPU)
  first      global index of the call's first sample
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2512_20064_amd import mps, synth

DEV = "cuda"


def _case(name, call="sample", precision="fp32", M=16, d=4, chi=64, N=1024, **more):
    c = {"name": name, "call": call, "precision": precision, "M": M, "M_hi": M, "d": d, "d_hi": d, "chi": chi,
         "N": N, "B": 1, "sigma": 0.0, "storage": "c64", "host": False, "first": 0}
    c.update(more)
    return c


def listed():
    return [
        # the smallest call: a handful of samples of a short qubit chain (latency of one launch and the call's host path)
        _case("tiny_fp32", M=8, d=2, chi=8, N=64),
        # the parity configuration of the benchmark: a small chain, one persistent launch
        _case("small_fp32", M=32, d=4, chi=32, N=4096),
        # a few hundred samples in the headline form: launches and their gaps
        _case("few_fp16f6", precision="fp16f6", M=24, d=4, chi=64, N=512),
        # bonds that are no multiple of any tile, an odd sample count, not the first rank of a sharded job
        _case("ragged_bf16x3", precision="bf16x3", M=40, d=3, chi=100, N=2999, first=4099),
        # one chain of a medium ensemble in the reference precision
        _case("medium_fp32", M=48, d=3, chi=256, N=8192),
        # an ensemble of chains of different lengths and bonds in one batched call
        _case("ensemble_fp16f8", call="batch", precision="fp16f8", M=32, M_hi=96, d=2, d_hi=4, chi=256, N=2048, B=24),
        # a window of the headline chain: one full chunk at chi = 1024
        _case("plateau_fp16f6", precision="fp16f6", M=22, d=4, chi=1024, N=65536),
        # the same chain in plain FP32, a smaller macro batch
        _case("plateau_fp32", M=18, d=4, chi=1024, N=16384),
        # and in the split 16-bit form, a macro batch that is no multiple of a tile
        _case("plateau_bf16x3", precision="bf16x3", M=18, d=4, chi=1024, N=20000),
        # the boson-sampling variant: every sample displaces every site
        _case("displaced_fp16f6", precision="fp16f6", M=18, d=4, chi=1024, N=32768, sigma=0.5),
        # a chain whose physical dimension varies, bonds in the thousands, a macro batch of 8192
        _case("uneven_fp16f6", precision="fp16f6", M=18, d=2, d_hi=6, chi=4096, N=8192),
        # site tensors streamed from pinned host memory as complex-fp16
        _case("streamed_fp16x3", call="stored", precision="fp16x3", M=16, d=4, chi=2048, N=16384, storage="cf16",
              host=True),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


# Algorithmic TFLOP/s of the forms on the plateau; with 20 us a site, what a drawn case may cost.
_RATE = {"fp32": 100e12, "bf16x3": 400e12, "fp16x3": 400e12, "fp16f8": 500e12, "fp16f6": 560e12}
_MOST_S = 0.04


def _cost(c):
    chains = _plan(c)
    per_row = sum(8.0 * chi[k] * d[k] * chi[k + 1] for d, chi in chains for k in range(len(d)))
    sites = max(len(d) for d, _ in chains)
    return c["N"] * per_row / _RATE[c["precision"]] * (1.4 if c["sigma"] else 1.0) + 20e-6 * sites


def draw(rng):
    """One more case of the same ranges: sizes over their logarithm, odd ones among them."""
    call = rng.choice(["sample", "sample", "sample", "batch", "stored"])
    precision = rng.choice(["fp32", "fp16f6", "fp16f6", "fp16f8", "bf16x3", "fp16x3"])
    d = rng.randint(2, 4)
    c = _case(None, call=call, precision=precision, M=_log_int(rng, 6, 48), d=d, chi=_log_int(rng, 8, 2048),
              N=_log_int(rng, 32, 65536), d_hi=d, first=rng.choice([0, 0, rng.randint(1, 10 ** 9)]))
    del c["name"]
    if rng.random() < 0.3:
        c["d_hi"] = rng.randint(d, 6)
    c["M_hi"] = c["M"]
    if call == "batch":
        c.update(B=rng.randint(2, 24), chi=_log_int(rng, 16, 256), N=_log_int(rng, 32, 8192),
                 M_hi=c["M"] + rng.randint(0, 64))
    elif call == "stored":
        c.update(storage=rng.choice(["cf16", "cf8"]), host=rng.random() < 0.7)
    if call != "batch" and rng.random() < 0.25:
        c["sigma"] = round(rng.uniform(0.1, 0.8), 3)
    while _cost(c) > _MOST_S and c["N"] > 32:
        c["N"] = max(32, int(c["N"] * 0.7))
    return c


# ---- chains ------------------------------------------------------------------

def _plan(c):
    """(d_k, chi_k) of the case's chains: shapes depend on the case alone."""
    rng = np.random.Generator(np.random.PCG64([c["M"], c["d"], c["d_hi"], c["chi"], c["B"]]))
    out = []
    for _ in range(c["B"]):
        if c["call"] == "batch":
            M = int(rng.integers(c["M"], c["M_hi"] + 1))
            d = [int(rng.integers(c["d"], c["d_hi"] + 1))] * M
            caps = [x for x in (16, 32, 64, 128, 256) if x <= c["chi"]] or [c["chi"]]
            cap = int(rng.choice(sorted(set(caps + [c["chi"]]))))
        else:
            M, cap = c["M"], c["chi"]
            d = [int(x) for x in rng.integers(c["d"], c["d_hi"] + 1, size=M)]
        out.append((d, synth.ramp_bonds(d, cap)))
    return out


def _dense_site(gen, chi_l, d, chi_r):
    """Random right-canonical complex64 site (decaying branch weights), made on
    the GPU: G with rows made orthonormal by the Cholesky factor of G G^H."""
    G = torch.randn((chi_l, d, chi_r), dtype=torch.complex128, device=DEV, generator=gen)
    G = G * torch.exp(-0.5 * torch.arange(d, device=DEV, dtype=torch.float64))[None, :, None]
    G = G.reshape(chi_l, d * chi_r)
    L = torch.linalg.cholesky(G @ G.conj().T.contiguous())
    return torch.linalg.solve_triangular(L, G, upper=False).to(torch.complex64).reshape(chi_l, d, chi_r).contiguous()


def _chain(c, b, d, chi, seed):
    """The chain's site tensors: dense random sites, one buffer per site, up to
    a bond of 1024; the structured sites of the large-bond workloads above
    (repeated shapes share a buffer).  A repeated shape cycles over 3 tensors."""
    if max(chi) > 1024:
        return synth.structured_chain(seed * 64 + b, d, max(chi), pool=2, device=DEV)[0]
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed * 1000 + b)
    pool, seen, out = {}, {}, []
    for k in range(len(d)):
        shape = (chi[k], d[k], chi[k + 1])
        seen[shape] = seen.get(shape, 0) + 1
        key = shape + (seen[shape] % 3,)
        if key not in pool:
            pool[key] = _dense_site(gen, *shape)
            out.append(pool[key])
        else:
            out.append(pool[key].clone())
    return out


def _displacements(c, seed):
    if not c["sigma"]:
        return None
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed * 7 + 3)
    return (c["sigma"] * torch.randn((c["N"], c["M"]), dtype=torch.complex64, device=DEV, generator=gen)).contiguous()


def _inputs(c, seed):
    plan = _plan(c)
    sites = [_chain(c, b, d, chi, seed) for b, (d, chi) in enumerate(plan)]
    return plan, sites, _displacements(c, seed)


# ---- what is measured ----------------------------------------------------------

def prepare(case, seed):
    plan, sites, mu = _inputs(case, seed)
    s = {"call": case["call"], "N": case["N"], "first": case["first"], "seed": seed + 17, "mu": mu,
         "sampler": mps.Sampler(0, precision=case["precision"])}
    if case["call"] == "batch":
        s["batch"] = mps.prepare_batch(sites)
    elif case["call"] == "stored":
        raw = {}
        for t in sites[0]:
            if id(t) not in raw:
                r = synth.compress_site_torch(t, case["storage"])
                raw[id(t)] = r.cpu().pin_memory() if case["host"] else r
        s.update(stored=[raw[id(t)] for t in sites[0]], shapes=[tuple(t.shape) for t in sites[0]],
                 kind=case["storage"])
    else:
        s["sites"] = sites[0]
    torch.cuda.synchronize()
    return s


def run(state):
    s = state["sampler"]
    if state["call"] == "batch":
        return s.sample_batch(state["batch"], state["N"], state["seed"], n_offset=state["first"])
    if state["call"] == "stored":
        r = s.sample_stored(state["stored"], state["shapes"], state["kind"], state["N"], state["seed"],
                            n_offset=state["first"], displace=state["mu"])
    else:
        r = s.sample(state["sites"], state["N"], state["seed"], n_offset=state["first"], displace=state["mu"])
    return {"outcomes": r["outcomes"], "logp": r["logp"]}


def work(case):
    nbytes = flops = 0.0
    for d, chi in _plan(case):
        for k in range(len(d)):
            flops += 8.0 * case["N"] * chi[k] * d[k] * chi[k + 1]
            nbytes += synth.compressed_bytes(chi[k], d[k], chi[k + 1], case["storage"])
        nbytes += case["N"] * (4.0 * len(d) + 8.0)
        if case["sigma"]:
            nbytes += 8.0 * case["N"] * len(d)
    return {"bytes": nbytes, "flops": flops}


# ---- the same in 64 bits ---------------------------------------------------------

_W = 0xFFFFFFFFFFFFFFFF


def _mul128(a, m):
    """High and low words of a * m, a an array of uint64."""
    lo = a * np.uint64(m)
    a0, a1 = a & np.uint64(0xFFFFFFFF), a >> np.uint64(32)
    m0, m1 = np.uint64(m & 0xFFFFFFFF), np.uint64(m >> 32)
    t = a1 * m0 + ((a0 * m0) >> np.uint64(32))
    u = a0 * m1 + (t & np.uint64(0xFFFFFFFF))
    return a1 * m1 + (t >> np.uint64(32)) + (u >> np.uint64(32)), lo


def _uniforms(seed, mps_id, first, N, k):
    """First word of Philox4x64-10 (Salmon et al. 2011) at counter (sample, site), key (seed, chain), as a uniform."""
    x = [np.arange(first, first + N, dtype=np.uint64), np.full(N, k, np.uint64), np.zeros(N, np.uint64),
         np.zeros(N, np.uint64)]
    a, b = seed, mps_id
    for _ in range(10):
        h0, l0 = _mul128(x[0], 0xD2E7470EE14C6C93)
        h1, l1 = _mul128(x[2], 0xCA5A826395121157)
        x = [h1 ^ x[1] ^ np.uint64(a), l1, h0 ^ x[3] ^ np.uint64(b), l0]
        a, b = (a + 0x9E3779B97F4A7C15) & _W, (b + 0xBB67AE8584CAA73B) & _W
    return torch.from_numpy(((x[0] >> np.uint64(12)).astype(np.float64) + 0.5) * 2.0 ** -52).to(DEV)


def _decode(raw, shape, kind):
    """complex128 site from its stored bytes."""
    n = shape[0] * shape[1] * shape[2]
    if kind == "cf16":
        ri = raw[:4 * n].view(torch.float16).to(torch.float64).reshape(*shape, 2)
        return torch.view_as_complex(ri.contiguous())
    ncol = shape[1] * shape[2]
    ri = raw[:2 * n].view(torch.float8_e4m3fn).to(torch.float64).reshape(shape[0], ncol, 2)
    nbr, nbc = -(-shape[0] // 128), -(-ncol // 128)
    off = -(-2 * n // 256) * 256
    sc = raw[off:off + 4 * nbr * nbc].view(torch.float32).to(torch.float64).reshape(nbr, nbc)
    sc = sc.repeat_interleave(128, 0).repeat_interleave(128, 1)[:shape[0], :ncol]
    return torch.view_as_complex((ri * sc[:, :, None]).contiguous()).reshape(shape)


def _operators(mu, d):
    """exp(-|mu|^2/2) exp(mu a^+) exp(-mu^* a) on d levels, one per sample (both exponents are nilpotent)."""
    a = torch.diag(torch.sqrt(torch.arange(1, d, dtype=torch.float64)), 1).to(torch.complex128).to(DEV)
    up, down = mu[:, None, None] * a.T.contiguous(), -mu.conj()[:, None, None] * a
    eye = torch.eye(d, dtype=torch.complex128, device=DEV).expand(mu.numel(), d, d)
    eu, ed, pu, pd = eye.clone(), eye.clone(), eye.clone(), eye.clone()
    mul = lambda x, y: (x[:, :, :, None] * y[:, None, :, :]).sum(2)  # noqa: E731
    for k in range(1, d):
        pu, pd = mul(pu, up) / k, mul(pd, down) / k
        eu, ed = eu + pu, ed + pd
    return torch.exp(-mu.abs() ** 2 / 2)[:, None, None] * mul(eu, ed)


def _sweep64(site, d, chi, N, seed, mps_id, first, mu):
    """logp of N samples drawn in 64 bits; site(k): complex128 tensor (chi_k, d_k, chi_{k+1})."""
    logp = torch.zeros(N, dtype=torch.float64, device=DEV)
    step = max(256, int(2 ** 31 / (16 * max(d[k] * chi[k + 1] for k in range(len(d))))))
    left = [torch.ones((min(step, N - r), 1), dtype=torch.complex128, device=DEV) for r in range(0, N, step)]
    for k in range(len(d)):
        A = site(k).reshape(chi[k], -1)
        u = _uniforms(seed, mps_id, first, N, k)
        for i, r in enumerate(range(0, N, step)):
            rows = slice(r, min(N, r + step))
            W = (left[i] @ A).reshape(-1, d[k], chi[k + 1])
            if mu is not None:
                D = _operators(mu[rows, k].to(torch.complex128), d[k])
                W = sum(D[:, :, j, None] * W[:, j, None, :] for j in range(d[k]))
            q = torch.view_as_real(W).square().sum((2, 3))
            P = torch.cumsum(q, 1)
            S = P[:, -1]
            s = (u[rows, None] > P / S[:, None]).sum(1).clamp(max=d[k] - 1)
            at = torch.arange(s.numel(), device=DEV)
            qs = q[at, s]
            logp[rows] += torch.log(qs / S)
            left[i] = W[at, s] / torch.sqrt(qs)[:, None]
    return logp


def exact(case, seed):
    """The log-probabilities of the samples as 64-bit arithmetic draws them (outcomes are whole numbers: none)."""
    if case["N"] * sum(8.0 * chi[k] * d[k] * chi[k + 1] for d, chi in _plan(case) for k in range(len(d))) > 60e12:
        return None
    plan, sites, mu = _inputs(case, seed)
    out = []
    for b, (d, chi) in enumerate(plan):
        if case["call"] == "stored":
            raw = {id(t): (synth.compress_site_torch(t, case["storage"]), tuple(t.shape)) for t in sites[b]}
            site = lambda k: _decode(*raw[id(sites[b][k])], case["storage"])  # noqa: E731
        else:
            site = lambda k: sites[b][k].to(torch.complex128)  # noqa: E731
        out.append((None, _sweep64(site, d, chi, case["N"], seed + 17, b, case["first"], mu)))
    return out if case["call"] == "batch" else {"outcomes": None, "logp": out[0][1]}
