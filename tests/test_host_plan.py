"""Planning in the C ABI's host code (routes, scratch, launches, messages), run
on the CPU: mps_abi.cpp linked with a stand-in for the HIP runtime and the
kernel launches (host_hip.cpp), which logs every launch."""
import ctypes
import os
import re
import shutil
import subprocess

import pytest

from paper_2512_20064_amd import build, mps, synth

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def host_lib(tmp_path_factory):
    cc = build.hipcc()
    if shutil.which(cc) is None and not os.path.exists(cc):
        pytest.skip("no hipcc")
    d = tmp_path_factory.mktemp("host")
    objs = []
    for src in (os.path.join(build.CSRC, "mps_abi.cpp"), os.path.join(HERE, "host_hip.cpp")):
        objs.append(str(d / (os.path.basename(src) + ".o")))
        subprocess.run([cc, "-O1", "-std=c++17", f"--offload-arch={build.ARCH}", "-fPIC",
                        "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                        "-x", "hip", "-c", src, "-o", objs[-1]], check=True, capture_output=True)
    lib = str(d / "libmps_host.so")
    # (-Bsymbolic: a HIP runtime that torch has loaded does not come first)
    subprocess.run(["g++", "-shared", "-Wl,-Bsymbolic", *objs, "-lpthread", "-o", lib], check=True,
                   capture_output=True)
    return lib


@pytest.fixture
def host(host_lib, monkeypatch):
    monkeypatch.setattr(mps, "_lib", None)
    lib = mps.load(host_lib)
    lib.host_log.restype = ctypes.c_char_p
    lib.host_peak.restype = ctypes.c_size_t
    lib.host_reset.argtypes = [ctypes.c_size_t]
    lib.host_set_pinned.argtypes = [ctypes.c_void_p, ctypes.c_void_p]
    lib.host_reset(1 << 40)
    return lib


def _log(lib):
    """The launches since the last call, [(kind, {field: value})]."""
    out = [(ln.split()[0], {k: int(v) for k, v in re.findall(r"(\w+)=(\d+)", ln)})
           for ln in lib.host_log().decode().splitlines()]
    lib.host_clear_log()
    return out


def _handle(precision, **kw):
    o = mps.mps_options_init()
    o.precision = mps.PRECISIONS[precision]
    for k, v in kw.items():
        setattr(o, k, v)
    return mps.mps_create(0, o), o


def _sites(M):
    """Site pointers that are never read (device memory, extent unknown)."""
    return [0x10000000 + 0x1000 * k for k in range(M)]


def _sample(h, chi, d, N):
    M = len(d)
    return mps.mps_sample(h, _sites(M), mps.MPS_C64, chi, d, M, N, 0, 1, 0x1000, 0)


def _autotune(h, chi, d, N, tensors=None):
    M = len(d)
    return mps.mps_autotune(h, tensors or _sites(M), mps.MPS_C64, chi, d, M, N, 1)


# one warm-up and three timed sweeps of a candidate
SWEEPS = 4


@pytest.mark.parametrize("form,d,cap,kind", [
    ("bf16x3", [4] * 16, 128, "mid"),
    ("fp16f6", [4] * 16, 256, "mid"),
    ("fp32", [2] * 16, 100, "mid"),
    ("fp32", [4] * 12, 32, "small"),
    ("fp16f8", [4] * 12, 32, "small"),
    ("fp32", [4] * 16, 256, "contract"),
])
def test_autotune_times_the_chain_in_every_candidate(host, form, d, cap, kind):
    """Every timed sweep of every candidate launches the probe's sites."""
    chi = synth.ramp_bonds(d, cap)
    h, _ = _handle(form)
    rc, rep = _autotune(h, chi, d, 40000)
    assert rc == 0, mps.mps_last_error()
    log = [x for x in _log(host) if x[0] == kind]
    sites = rep.probe_sites if kind == "contract" else 1
    for rows in (8192, 16384, 32768, 40000):
        n = sum(f["rows"] == rows for _, f in log)
        assert n >= SWEEPS * sites and n % (SWEEPS * sites) == 0, (rows, n)
    assert rep.candidates == 16 and rep.skipped == 0
    mps.mps_destroy(h)


def _plateau(M, d, chi):
    return synth.ramp_bonds([d] * M, chi)


@pytest.mark.parametrize("name,form,chi,d,want", [
    # packed sites of the whole chain above the limit of the persistent kernel
    ("packed", "bf16x3", _plateau(600, 4, 256), [4] * 600, "contract"),
    ("fits", "bf16x3", _plateau(60, 4, 256), [4] * 60, "mid"),
    # the largest site lies in a small-bond prefix, a bond of 33 follows
    ("wider later", "bf16x3", [1, 4, 16, 32, 32, 16, 33, 33, 33], [4, 4, 4, 4, 2, 4, 2, 1], "mid"),
    ("wider later", "fp16", [1, 4, 16, 32, 32, 16, 33, 33, 33], [4, 4, 4, 4, 2, 4, 2, 1], "contract"),
    # displaced, or some later site in host memory: per site
    ("displaced", "fp16f6", _plateau(16, 4, 64), [4] * 16, "contract"),
    ("displaced", "fp32", _plateau(12, 4, 16), [4] * 12, "contract"),
    ("pinned tail", "fp16f6", _plateau(16, 4, 64), [4] * 16, "contract"),
])
def test_autotune_probe_takes_the_kernels_of_the_job(host, name, form, chi, d, want):
    M, N = len(d), 20000
    h, o = _handle(form, displace=0x1000 if name == "displaced" else None)
    sites = _sites(M)
    if name == "pinned tail":
        host.host_set_pinned(sites[-1], sites[-1] + 1)
    rc, rep = _autotune(h, chi, d, N, sites)
    assert rc == 0, mps.mps_last_error()
    log = _log(host)
    kinds = {k for k, _ in log} & {"small", "mid", "contract"}
    assert kinds == {want} and rep.candidates == 12 and rep.probe_sites < M
    if want != "contract":  # no tile order to time: once per chunk, the default kept
        for rows in (8192, 16384, 20000):
            assert sum(k == want and f["rows"] == rows for k, f in log) == SWEEPS
        assert rep.tile_group == 4
    if name in ("packed", "fits", "displaced"):  # and it is the job's own route
        if name == "displaced":
            o.displace = 0x1000
            mps.mps_set_options(h, o)
        assert _sample(h, chi, d, 100) == 0, mps.mps_last_error()
        assert {k for k, _ in _log(host)} & {"small", "mid", "contract"} == {want}
    mps.mps_destroy(h)


def _batch(h, shapes, N):
    """mps_sample_batch over chains of (chi, d); pointers are never read."""
    descs, keep = [], []
    for b, (chi, d) in enumerate(shapes):
        c, k = mps.make_chain(_sites(len(d)), chi, d, b, 0x1000, None)
        descs.append(c)
        keep.append(k)
    return mps.mps_sample_batch(h, descs, mps.MPS_C64, N, 0, 1)


@pytest.mark.parametrize("form", ["fp32", "bf16x3", "fp16f6"])
@pytest.mark.parametrize("B,M,N", [(100, 8, 64), (300, 4, 10), (1, 4, 1), (3, 30, 500)])
def test_scratch_stays_under_the_cap(host, form, B, M, N):
    """Whatever route a call takes, the memory it allocates stays within
    max_device_bytes, and the caps and chunks that are accepted are those of
    the per-site launches."""
    d = [4] * M
    chi = [1, 4, 16, 40] + [40] * (M - 3)
    routes = set()
    for i in range(70):
        cap = int(20000 * 1.2 ** i)
        got = []
        for fused in (0, 1):
            host.host_reset(1 << 40)
            h, _ = _handle(form, max_device_bytes=cap, fused_small=fused)
            rc = _batch(h, [(chi, d)] * B, N)
            got.append((rc, mps.mps_get_stats(h).n_chunk))
            assert host.host_peak() <= cap, (cap, host.host_peak())
            routes |= {k for k, _ in _log(host)}
            mps.mps_destroy(h)
        assert got[0] == got[1], (cap, got)
    assert {"mid", "contract"} <= routes


@pytest.mark.parametrize("form,cap,d", [
    ("fp32", 8, 2), ("fp32", 64, 4), ("fp16f6", 100, 3), ("bf16x3", 300, 4),
])
def test_flagged_samples_are_counted_out_of_all(host, form, cap, d):
    """The message of MPS_ENUMERIC names the samples of every chain of the
    call, whatever kernels the chains take."""
    dl = [d] * 9
    chi = synth.ramp_bonds(dl, cap)
    h, _ = _handle(form)
    host.host_set_flagged(7)
    assert _sample(h, chi, dl, 400) == mps.MPS_ENUMERIC
    assert mps.mps_last_error().startswith("7 of 400 samples"), mps.mps_last_error()
    assert _batch(h, [(chi, dl), ([1, 2, 1], [2, 2]), (chi, dl)], 50) == mps.MPS_ENUMERIC
    assert mps.mps_last_error().startswith("7 of 150 samples"), mps.mps_last_error()
    mps.mps_destroy(h)


@pytest.mark.parametrize("form,d,chi,B,N,n_chunk", [
    ("fp32", [2], [1, 1], 1, (1 << 28) + 5, 1 << 29),              # small-bond kernel: 16 samples a workgroup
    ("fp32", [2, 2], [1, 2, 1], 5000, 65536, 0),
    ("fp16f6", [2], [1, 1], 20000, 1 << 21, 1 << 21),              # more than 2^31 workgroups in one launch
    ("bf16x3", [5, 1], [1, 5, 5], 1, (1 << 28) + 5, 1 << 29),      # medium-bond kernel, 8 waves
    ("fp16f6", [3, 1], [1, 40, 40], 1, (1 << 29) + 5, 1 << 30),    # and 4
])
def test_large_launches_stay_within_the_grid(host, form, d, chi, B, N, n_chunk):
    """Chunks whose persistent launch would have 2^32 threads or more (HIP
    refuses those) are cut, or the chain takes the per-site launches."""
    host.host_reset(1 << 46)
    h, _ = _handle(form, n_chunk=n_chunk)
    desc, keep = mps.make_chain(_sites(len(d)), chi, d, 0, 0x1000, None)
    descs = (mps.mps_chain * B)(*[desc] * B)
    rc = host.mps_sample_batch(h, B, descs, mps.MPS_C64, N, 0, ctypes.c_uint64(1))
    assert rc == 0, mps.mps_last_error()
    log = _log(host)
    done = [f["rows"] for k, f in log if k in ("small", "mid")] or \
        [f["rows"] for k, f in log if k == "measure"][::len(d)]
    assert sum(done) == N
    mps.mps_destroy(h)


@pytest.mark.parametrize("form", ["bf16x3", "fp16f6"])
def test_medium_bond_call_falls_back_when_memory_is_short(host, form):
    """A call whose packed sites do not fit in the memory that is left takes
    the per-site launches, which need one packed site at a time."""
    d, chi = [4] * 400, synth.ramp_bonds([4] * 400, 128)
    for limit, want in ((1 << 26, "contract"), (1 << 30, "mid"), (1 << 26, "contract")):
        host.host_reset(limit)
        h, _ = _handle(form)
        n0 = host.host_mallocs()
        for _ in range(3):
            assert _sample(h, chi, d, 16) == 0, mps.mps_last_error()
            assert {k for k, _ in _log(host)} & {"mid", "contract"} == {want}
        assert host.host_mallocs() == n0 + 1  # the scratch is kept from call to call
        host.host_reset(1 << 30)  # memory is free again: the same handle
        assert _sample(h, chi, d, 16) == 0, mps.mps_last_error()
        assert {k for k, _ in _log(host)} & {"mid", "contract"} == {"mid"}
        mps.mps_destroy(h)
    host.host_reset(1 << 20)  # too little for either
    h, _ = _handle(form)
    assert _sample(h, chi, d, 16) == mps.MPS_ENOMEM
    mps.mps_destroy(h)
