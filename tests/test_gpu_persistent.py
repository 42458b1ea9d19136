"""Routes to and around the persistent kernels: flagged samples and entries that
are not finite, chunked, captured, capped and allocation-free calls, batches
with a chain that fits no persistent kernel, launches of 2^28 samples; bits
and statistics against the per-site launches."""
import numpy as np
import pytest

from paper_2512_20064_amd import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SPLIT = ["fp16f6", "fp16f8", "bf16x3", "fp16x3"]


def _chain(seed, d, cap):
    return synth.to_c64(synth.random_mps(seed, d, synth.ramp_bonds(d, cap)))


def _same(a, b, msg=""):
    for key in ("outcomes", "logp", "probs", "u"):
        if key in a:
            assert np.array_equal(a[key].cpu().numpy(), b[key].cpu().numpy(), equal_nan=True), (key, msg)


def _forked(seed, d, cap, k, kind):
    """A chain whose site k - 1 sends outcome 0 to the first half of bond k and
    the others to the second; site k is zero, overflows or is not finite where
    the first half meets it."""
    t = _chain(seed, d, cap)
    h = t[k].shape[0] // 2
    t[k - 1][:, 0, h:] = 0
    t[k - 1][:, 1:, :h] = 0
    if kind == "zero":
        t[k][:h] = 0
    elif kind == "over":
        t[k][:h] = 3e38
    else:
        t[k][0, 0, 0] = complex(float(kind), 0)
    return t


@pytest.mark.parametrize("kind", ["zero", "over", "nan", "inf"])
@pytest.mark.parametrize("d,cap", [(2, 50), (2, 128), (4, 100), (4, 250)])
@pytest.mark.parametrize("form", ["fp32"] + SPLIT)
def test_flagged_samples_beside_live_ones(form, d, cap, kind):
    """Samples flagged in mid-chain, with live ones in the same workgroup (or
    all of them, for an entry that is not finite): the bits, the count and the
    status of the per-site launches."""
    from paper_2512_20064_amd import mps
    from tests.parity_util import EPS_FP32, EPS_LOWP, compare, upload
    print(f"[gpu-case] flagged {form} d={d} cap={cap} {kind}", flush=True)
    dl = [d] * 20
    t = _forked(5, dl, cap, 9, kind)
    dev = upload(t)
    N, seed = 70, 91
    a, b = mps.Sampler(0, precision=form), mps.Sampler(0, precision=form, fused_small=False)
    ra, rb = a.sample(dev, N, seed, emit_n=N), b.sample(dev, N, seed, emit_n=N)
    torch.cuda.synchronize()
    if form in SPLIT:
        assert a.stats.pack_launches == 1 and b.stats.pack_launches == 20
    elif d == 2:
        assert a.stats.scratch_bytes < b.stats.scratch_bytes  # no W in memory
    _same(ra, rb)
    assert ra["status"] == rb["status"] == mps.MPS_ENUMERIC
    assert a.stats.flagged == b.stats.flagged > 0
    o = ra["outcomes"].cpu().numpy()
    live = np.flatnonzero(o[:, -1] >= 0)
    assert len(live) == N - a.stats.flagged and (o[:, :9] >= 0).all()
    if kind == "zero":
        assert 0 < len(live) < N
        g = {"outcomes": o, "logp": ra["logp"].cpu().numpy(), "probs": ra["probs"].cpu().numpy(),
             "u": ra["u"].cpu().numpy()}
        compare(t, seed, g, rows=live, eps=EPS_FP32 if form == "fp32" else EPS_LOWP)
    elif kind == "over":
        assert len(live) < N and (len(live) > 0 or form not in ("fp32", "bf16x3"))
    else:
        assert len(live) == 0
    a.close()
    b.close()


@pytest.mark.parametrize("form,d,cap", [("fp32", 2, 100)] + [(f, 4, 100) for f in SPLIT] + [("fp16f6", 3, 33),
                                                                                           ("bf16x3", 4, 256)])
def test_ways_to_call_the_medium_bond_kernel(form, d, cap):
    """Chunks with a short last one, a captured graph, profiling, no logp, a
    first sample index, the allocation-free call, and caps on either side of
    what the kernel needs: the bits of the per-site launches."""
    from paper_2512_20064_amd import mps
    from tests.parity_util import upload
    print(f"[gpu-case] ways to call {form} d={d} cap={cap}", flush=True)
    dl = [d] * 13
    dev = upload(_chain(6, dl, cap))
    N, seed, first = 333, 17, 1 << 33
    ref = mps.Sampler(0, precision=form, fused_small=False)
    want = ref.sample(dev, N, seed, n_offset=first)
    torch.cuda.synchronize()
    per_site = ref.stats.scratch_bytes
    stream = torch.cuda.Stream()

    def persistent(st, chunks):
        if form == "fp32":
            return st.scratch_bytes < per_site
        return st.pack_launches == 1 and st.contract_launches == len(dl) * chunks

    s = mps.Sampler(0, precision=form)
    r = s.sample(dev, N, seed, n_offset=first)
    torch.cuda.synchronize()
    _same(r, want, "plain")
    assert persistent(s.stats, 1)
    need = s.stats.scratch_bytes
    s.close()

    s = mps.Sampler(0, precision=form, n_chunk=100, graph=True)
    for rep in range(3):
        torch.ones(1000, device="cuda").sum().item()  # eager work between the replays
        with torch.cuda.stream(stream):
            r = s.sample(dev, N, seed, n_offset=first, stream=stream)
        torch.cuda.synchronize()
        _same(r, want, f"graph {rep}")
        assert persistent(s.stats, 4) and s.stats.n_chunk == 100
    s.close()

    s = mps.Sampler(0, precision=form, n_chunk=128, profile=True)
    r = s.sample(dev, N, seed, n_offset=first, want_logp=False)
    torch.cuda.synchronize()
    assert torch.equal(r["outcomes"], want["outcomes"]) and r["logp"] is None
    assert persistent(s.stats, 3) and s.stats.contract_ms > 0
    assert s.stats.pack_ms > 0 or form == "fp32"
    s.close()

    # (in FP32 the kernel needs less than the smallest per-site plan, which has
    # to fit the cap whatever the route)
    for cap_bytes in (need, need - 1) if form != "fp32" else (per_site, 60000):
        s = mps.Sampler(0, precision=form, max_device_bytes=cap_bytes)
        r = s.sample(dev, N, seed, n_offset=first)
        torch.cuda.synchronize()
        _same(r, want, f"cap {cap_bytes}")
        assert s.stats.scratch_bytes <= cap_bytes
        s.close()

    o = mps.mps_options_init()
    o.precision = mps.PRECISIONS[form]
    h = mps.mps_create(0, o)
    chi = [1] + [int(x.shape[2]) for x in dev]
    for rep in range(2):
        out = torch.full((N, len(dl)), -7, dtype=torch.int32, device="cuda")
        lp = torch.full((N,), float("nan"), dtype=torch.float64, device="cuda")
        rc = mps.mps_sample_noalloc(h, [x.data_ptr() for x in dev], mps.MPS_C64, chi, dl, len(dl), N, first, seed,
                                    out.data_ptr(), lp.data_ptr())
        torch.cuda.synchronize()
        assert rc == 0, mps.mps_last_error()
        _same({"outcomes": out, "logp": lp}, want, f"noalloc {rep}")
        assert persistent(mps.mps_get_stats(h), 1)
    mps.mps_destroy(h)
    ref.close()


@pytest.mark.parametrize("form", ["fp32"] + SPLIT)
def test_batch_with_a_chain_that_fits_no_persistent_kernel(form):
    """With one such chain every chain of the batch takes the per-site launches;
    the bits of each are those of a call of its own."""
    from paper_2512_20064_amd import mps
    from tests.parity_util import upload
    print(f"[gpu-case] batch with a large chain {form}", flush=True)
    specs = [([2] * 12, 40), ([2] * 14, 100), ([3] * 8, 64), ([2] * 18, 300)]
    chains = [upload(_chain(50 + i, d, c)) for i, (d, c) in enumerate(specs)]
    for large in (False, True):
        use = chains if large else chains[:2]
        M = max(len(c) for c in use)
        s = mps.Sampler(0, precision=form, n_chunk=150)
        p = mps.Sampler(0, precision=form, n_chunk=150, fused_small=False)
        outs, per_site = s.sample_batch(use, 333, 5), p.sample_batch(use, 333, 5)
        torch.cuda.synchronize()
        if form in SPLIT:
            assert s.stats.pack_launches == (3 * M if large else 1)
        assert (s.stats.scratch_bytes == p.stats.scratch_bytes) == large or form in SPLIT
        for i in range(len(use)):
            one = mps.Sampler(0, precision=form, mps_id=i)
            r = one.sample(use[i], 333, 5)
            torch.cuda.synchronize()
            for o, lp in (outs[i], per_site[i]):
                assert torch.equal(o, r["outcomes"]) and torch.equal(lp, r["logp"]), (i, large)
            one.close()
        s.close()
        p.close()


@pytest.mark.parametrize("form", ["fp32", "bf16x3", "fp16f6"])
def test_tile_choices_of_a_batch_on_the_per_site_launches(form):
    """Wide, narrow and mixed tiles of the steps of a batch give the same bits
    (fused_small off: the persistent kernels have no tiles)."""
    from paper_2512_20064_amd import mps
    from tests.parity_util import upload
    print(f"[gpu-case] batch tiles {form}", flush=True)
    specs = [([2, 3, 4, 4, 3, 2, 2], 64), ([4] * 8, 96), ([3] * 9, 160), ([2, 2, 4, 4, 4, 2], 48)]
    chains = [upload(_chain(60 + i, d, c)) for i, (d, c) in enumerate(specs)]
    N, seed = 700, 3
    shapes = sorted({tuple(int(n) for n in x.shape) for c in chains for x in c})
    s = mps.Sampler(0, precision=form, n_chunk=N, fused_small=False)
    runs = []
    for pick in (lambda i: 0, lambda i: 1, lambda i: i % 2):
        s.set_tiles([])
        s.set_tiles([dict(chi_l=a, d=b, chi_r=c, tile=pick(i), rows=N) for i, (a, b, c) in enumerate(shapes)])
        runs.append(s.sample_batch(chains, N, seed))
        torch.cuda.synchronize()
        assert s.stats.contract_launches == 9
    for other in runs[1:]:
        for (o1, l1), (o2, l2) in zip(runs[0], other):
            assert torch.equal(o1, o2) and torch.equal(l1, l2)
    s.close()


@pytest.mark.parametrize("form,d,cap", [("bf16x3", 4, 128), ("fp32", 2, 100), ("fp16f6", 4, 16)])
def test_autotune_runs_the_probe_to_the_end(form, d, cap):
    """The last timed sweep of the autotuner ran the probe's sites."""
    from paper_2512_20064_amd import mps
    from tests.parity_util import upload
    print(f"[gpu-case] autotune probe {form} d={d} cap={cap}", flush=True)
    ch = upload(_chain(12, [d] * 16, cap))
    s = mps.Sampler(0, precision=form)
    rep = s.autotune(ch, 20000, seed=1)
    st = mps.mps_get_stats(s.h)
    assert st.n_chunk == 20000 and rep["candidates"] == 12 and rep["tile_group"] == 4
    if cap <= 32:
        assert st.fused_launches == 1 and st.fused_flops > 0
    else:
        assert st.contract_launches == rep["probe_sites"] and st.contract_flops > 0
    s.close()


def test_small_bond_launch_of_more_than_2_28_samples():
    """One chunk of 2^28 + 33 samples is cut where HIP's grid ends."""
    from paper_2512_20064_amd import mps
    print("[gpu-case] small-bond launch of 2^28 + 33 samples", flush=True)
    N = (1 << 28) + 33
    t = [torch.tensor([[[0.6], [0.8j]]], dtype=torch.complex64, device="cuda")]
    got = []
    for n_chunk in (1 << 29, 1 << 24):
        s = mps.Sampler(0, n_chunk=n_chunk)
        r = s.sample(t, N, 3, want_logp=False)
        torch.cuda.synchronize()
        got.append(r["outcomes"])
        assert s.stats.n_chunk <= n_chunk and s.stats.fused_launches == -(-N // s.stats.n_chunk)
        s.close()
    assert torch.equal(got[0], got[1])
    assert abs(got[0].float().mean().item() - 0.64) < 1e-3


@pytest.mark.parametrize("form,d,cap", [("fp32", 4, 32), ("fp32", 3, 27), ("fp32", 2, 16), ("fp32", 2, 100),
                                        ("fp32", 3, 45), ("fp16f6", 4, 100), ("bf16x3", 3, 65)])
def test_site_tensors_eight_bytes_off(form, d, cap):
    """Site tensors that start and end in the middle of 16 bytes: the bits of
    aligned ones."""
    from paper_2512_20064_amd import mps
    from tests.parity_util import upload
    print(f"[gpu-case] sites 8 bytes off {form} d={d} cap={cap}", flush=True)
    dev = upload(_chain(7, [d] * 9, cap))
    off = []
    for x in dev:
        buf = torch.full((x.numel() + 2,), float("nan"), dtype=torch.complex64, device="cuda")
        buf[1:-1] = x.reshape(-1)
        off.append(buf[1:-1].view(x.shape))
    assert all(x.data_ptr() % 16 == 8 for x in off)
    s = mps.Sampler(0, precision=form)
    a, b = s.sample(dev, 77, 5, emit_n=77), s.sample(off, 77, 5, emit_n=77)
    torch.cuda.synchronize()
    _same(a, b)
    s.close()
