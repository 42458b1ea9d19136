"""Sizes at the edges of the kernels' tiles, against the FP64 oracle (forced
prefix): sample counts around a workgroup's rows, odd bonds and column counts,
chains around the blocks in which uniforms and outcomes are handled."""
import pytest

from paper_2512_20064_amd import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SMALL = [
    # (d_k, chi_k, N, first sample)
    ([1], [1, 1], 1, 0),
    ([2] * 16, synth.ramp_bonds([2] * 16, 8), 15, 0),
    ([2] * 17, synth.ramp_bonds([2] * 17, 8), 17, 5),
    ([3, 4, 3, 4, 3, 4, 4], [1, 3, 11, 31, 29, 16, 4, 1], 50, 0),      # odd column counts, above and below 64
    ([4, 4, 4, 4, 2], [1, 4, 16, 27, 7, 5], 16, 1 << 33),             # an odd K, an open right end
    ([4] * 33, synth.ramp_bonds([4] * 33, 32), 33, 0),
]


def _check(t, s, N, first, eps):
    from tests.parity_util import compare, upload
    r = s.sample(upload(t), N, 77, n_offset=first, emit_n=N)
    torch.cuda.synchronize()
    g = {"outcomes": r["outcomes"].cpu().numpy(), "logp": r["logp"].cpu().numpy(),
         "probs": r["probs"].cpu().numpy(), "u": r["u"].cpu().numpy()}
    rep = compare(t, 77, g, n_offset=first, eps=eps)
    print(rep, flush=True)
    return g


@pytest.mark.parametrize("case", range(len(SMALL)))
def test_small_bond_kernel_edges(case):
    from paper_2512_20064_amd import mps
    from tests.parity_util import EPS_FP32
    d, chi, N, first = SMALL[case]
    print(f"[gpu-case] small-bond edges {case}: M={len(d)} N={N}", flush=True)
    t = synth.to_c64(synth.random_mps(41 + case, d, chi))
    s = mps.Sampler(0)
    _check(t, s, N, first, EPS_FP32)
    assert s.stats.fused_launches == 1 and s.stats.contract_launches == 0
    s.close()


# Medium-bond kernel: 4, 5, 8, 9 and 16 groups of 64 columns, bonds that are no
# multiple of 8, 16 or 64, more branches than a 4-wave workgroup has lanes for,
# sample counts around a workgroup's 32 rows, chains around a block of sites.
MID = [
    # (d_k, chi_k, N, first sample)
    ([4] * 9, [1, 4, 16, 64, 64, 64, 64, 16, 4, 1], 33, 0),
    ([2] * 8, [1, 2, 4, 8, 16, 32, 64, 65, 40], 31, 7),
    ([4, 4, 4, 3, 5, 4, 2], [1, 4, 16, 61, 97, 100, 50, 25], 70, 0),
    ([4] * 7, [1, 4, 16, 64, 128, 127, 33, 9], 64, 1 << 33),
    ([4] * 6, [1, 4, 16, 64, 256, 250, 63], 40, 0),
    ([10, 9, 3, 2], [1, 10, 60, 41, 21], 20, 0),
    ([16, 16, 2] + [1] * 15, [1, 16, 33, 40] + [40] * 15, 1, 3),
]


@pytest.mark.parametrize("form", ["fp16f6", "fp16f8", "bf16x3", "fp16x3"])
@pytest.mark.parametrize("case", range(len(MID)))
def test_medium_bond_kernel_edges(form, case):
    """The persistent kernel gives the bits of the per-site launches, and both
    agree with the oracle."""
    from paper_2512_20064_amd import mps
    from tests.parity_util import EPS_LOWP, upload
    d, chi, N, first = MID[case]
    print(f"[gpu-case] medium-bond edges {form} {case}: M={len(d)} N={N}", flush=True)
    t = synth.to_c64(synth.random_mps(61 + case, d, chi))
    a = mps.Sampler(0, precision=form)
    b = mps.Sampler(0, precision=form, fused_small=False)
    dev = upload(t)
    ra = a.sample(dev, N, 77, n_offset=first, emit_n=N)
    rb = b.sample(dev, N, 77, n_offset=first, emit_n=N)
    torch.cuda.synchronize()
    # packed in one launch for the call by the persistent kernel, in one per site otherwise
    assert a.stats.pack_launches == 1 and a.stats.contract_launches == len(d)
    assert b.stats.pack_launches == len(d) and b.stats.contract_launches == len(d)
    for key in ("outcomes", "logp", "u"):
        assert torch.equal(ra[key], rb[key]), key
    assert torch.equal(torch.nan_to_num(ra["probs"]), torch.nan_to_num(rb["probs"]))
    _check(t, a, N, first, EPS_LOWP)
    a.close()
    b.close()


@pytest.mark.parametrize("extra", [[], [([2] * 14, 300)]])
def test_medium_bond_kernel_batch_and_chunks(extra):
    """Chains of every kernel variant in one batched call with a ragged last
    chunk, without and with a chain that does not fit the kernel (all per-site
    then), against one call per chain on the per-site launches."""
    from paper_2512_20064_amd import mps
    from tests.parity_util import upload
    print("[gpu-case] medium-bond batch", flush=True)
    specs = [([4] * 5, 16), ([4] * 9, 64), ([3] * 11, 100), ([4] * 8, 200)] + extra
    chains = [upload(synth.to_c64(synth.random_mps(90 + i, d, synth.ramp_bonds(d, c)))) for i, (d, c) in
              enumerate(specs)]
    s = mps.Sampler(0, precision="fp16f6", n_chunk=100)
    outs = s.sample_batch(chains, 333, 5)
    torch.cuda.synchronize()
    for i, (o, lp) in enumerate(outs):
        one = mps.Sampler(0, precision="fp16f6", mps_id=i, fused_small=i == 0)
        r = one.sample(chains[i], 333, 5)
        torch.cuda.synchronize()
        assert torch.equal(o, r["outcomes"]) and torch.equal(lp, r["logp"]), i
        one.close()
    s.close()


@pytest.mark.parametrize("d,chi,N", [
    ([4] * 8, [1, 4, 16, 64, 130, 66, 34, 10, 4], 129),   # column and K tails of 2
    ([2, 4, 4, 6, 4, 2], [1, 2, 8, 32, 192, 62, 32], 127),
    ([4] * 6, [1, 4, 16, 63, 128, 65, 17], 200),           # odd bonds beside even ones
])
def test_fp32_direct_tile_edges(d, chi, N):
    """FP32 wide tile loaded straight into LDS: the bits of the register-staged
    narrow tile, also where a site starts 8 bytes off a 16-byte boundary (the
    register-staged wide tile), and the oracle."""
    from paper_2512_20064_amd import mps
    from tests.parity_util import EPS_FP32, upload
    print(f"[gpu-case] fp32 direct tile chi={chi} N={N}", flush=True)
    t = synth.to_c64(synth.random_mps(81, d, chi))
    s = mps.Sampler(0, fused_small=False)
    _check(t, s, N, 0, EPS_FP32)
    dev = upload(t)
    wide = s.sample(dev, N, 77)
    off = []
    for x in dev:
        buf = torch.empty(x.numel() + 1, dtype=torch.complex64, device="cuda")
        buf[1:] = x.reshape(-1)
        off.append(buf[1:].view(x.shape))
    assert all(x.data_ptr() % 16 == 8 for x in off)
    shifted = s.sample(off, N, 77)
    s.set_tiles([dict(chi_l=a, d=b, chi_r=c, tile=mps.MPS_TILE_NARROW, rows=N) for a, b, c in
                 {tuple(x.shape) for x in dev}])
    narrow = s.sample(dev, N, 77)
    torch.cuda.synchronize()
    for r in (shifted, narrow):
        assert torch.equal(r["outcomes"], wide["outcomes"]) and torch.equal(r["logp"], wide["logp"])
    s.close()


@pytest.mark.parametrize("d,chi,N,first", [
    ([4] * 9, [1, 4, 16, 64, 64, 61, 64, 16, 4, 1], 33, 0),        # 8 units, an odd bond
    ([2] * 18, [1, 2, 4, 8, 16, 32, 64, 65, 97, 128, 127, 90, 64, 32, 16, 8, 4, 2, 1], 31, 7),  # over a block of 16 sites
    ([3, 13, 2], [1, 3, 4, 2], 20, 0),                               # 26 units of small bonds: per site
    ([4, 4, 1, 1, 1, 1], [1, 4, 16, 16, 16, 16, 16], 1, 1 << 33),
    ([2, 2, 2, 2, 2, 2, 1], [1, 2, 4, 8, 16, 32, 50, 200], 70, 0),  # an open right end wider than the plateau
    ([8, 5, 1], [1, 8, 40, 41], 40, 0),                              # 16 and 10 units: per site
])
def test_fp32_medium_bond_kernel_edges(d, chi, N, first):
    """FP32: the persistent medium-bond kernel (where the chain's sites fit it)
    gives the bits of the per-site launches, and agrees with the oracle."""
    from paper_2512_20064_amd import mps
    from tests.parity_util import EPS_FP32, upload
    print(f"[gpu-case] fp32 medium-bond edges chi={chi} N={N}", flush=True)
    t = synth.to_c64(synth.random_mps(71, d, chi))
    small = max(chi) <= 32 and max(d) <= 4  # those take the small-bond kernel: other sums
    a, b = mps.Sampler(0), mps.Sampler(0, fused_small=False)
    dev = upload(t)
    ra = a.sample(dev, N, 77, n_offset=first, emit_n=N)
    rb = b.sample(dev, N, 77, n_offset=first, emit_n=N)
    torch.cuda.synchronize()
    if not small:
        if all(x * -(-c // 64) <= 4 for x, c in zip(d, chi[1:])):
            assert a.stats.scratch_bytes < b.stats.scratch_bytes  # no W in memory
        assert a.stats.contract_launches == b.stats.contract_launches == len(d)
        for key in ("outcomes", "logp", "probs", "u"):
            assert torch.equal(torch.nan_to_num(ra[key]), torch.nan_to_num(rb[key])), key
    _check(t, a, N, first, EPS_FP32)
    a.close()
    b.close()
