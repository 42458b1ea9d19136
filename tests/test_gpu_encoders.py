"""The operand encoders and turns of lp_ops.h on the GPU (e2m3_device.hip): the
E2M3 codes that the kernels form with the FP8 conversion instruction against
the definition e2m3_code (itself checked on the CPU), the turned operands and
the records of left vectors against numpy."""
import ctypes
import os

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

LIB = os.path.join(os.path.dirname(os.path.abspath(__file__)), "libe2m3_device.so")


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(LIB):
        from paper_2512_20064_amd import build
        build.build_checks()
    lib = ctypes.CDLL(LIB)
    P = ctypes.c_void_p
    lib.check_e2m3_codes.argtypes = [ctypes.c_uint32, ctypes.c_uint32, P]
    lib.turn_operands.argtypes = [P, P, ctypes.c_int]
    lib.split_slices.argtypes = [P, P, ctypes.c_int]
    torch.zeros(1, device="cuda")
    torch.cuda.synchronize()
    return lib


def _run(fn, *args):
    torch.cuda.synchronize()
    assert fn(*args) == 0
    torch.cuda.synchronize()


def test_conversion_codes_are_the_defined_ones(lib):
    """Every float of magnitude <= 7.5, in each position of the four."""
    print("[gpu-case] e2m3 codes of every float up to 7.5", flush=True)
    bad = torch.zeros(1, dtype=torch.int64, device="cuda")
    _run(lib.check_e2m3_codes, 0, 0x40F00001, bad.data_ptr())
    assert bad.item() == 0


def _pack6(codes):
    """32 codes of 6 bits -> 6 little-endian dwords."""
    v = sum(int(c) << (6 * p) for p, c in enumerate(codes))
    return [(v >> (32 * i)) & 0xFFFFFFFF for i in range(6)]


def test_turned_operands(lib):
    """(x, y) -> (-y, x) with the real parts in one half of a lane's values."""
    print("[gpu-case] turned operands", flush=True)
    n = 64
    rng = np.random.default_rng(7)
    inp, want = np.zeros((n, 20), np.uint32), np.zeros((n, 20), np.uint32)
    for t in range(n):
        e4 = rng.integers(0, 1 << 32, 8, dtype=np.uint32)
        c6 = rng.integers(0, 64, 32)
        scale = int(rng.integers(0, 256))
        h = rng.integers(0, 1 << 32, 4, dtype=np.uint32)
        inp[t] = [*e4, *_pack6(c6), scale, 0, *h]
        t4 = [x for i in range(0, 8, 2) for x in (e4[i + 1] ^ 0x80808080, e4[i])]
        want[t] = [*t4, *_pack6(np.concatenate([c6[16:] ^ 0x20, c6[:16]])), scale, 0,
                   h[2] ^ 0x80008000, h[3] ^ 0x80008000, h[0], h[1]]
    dev = torch.from_numpy(inp.view(np.int32)).cuda()
    out = torch.zeros_like(dev)
    _run(lib.turn_operands, dev.data_ptr(), out.data_ptr(), n)
    np.testing.assert_array_equal(out.cpu().numpy().view(np.uint32), want)


def _codes(x):
    """Nearest E2M3 codes of |x| <= 7.5, ties to the even mantissa."""
    a = np.abs(x)
    e = np.where(a < 1, 0, np.floor(np.log2(np.maximum(a, 1))))
    c = np.where(a < 1, np.rint(a * 8), (e + 1) * 8 + np.rint((a / 2.0 ** e - 1) * 8))
    return c.astype(np.int64) | np.where(np.signbit(x), 32, 0)


def test_records_of_left_vectors(lib):
    """split8_e2m3: fp16 parts, record scale and codes of slices of 8 complex
    whose magnitudes reach from 1 to below fp16's range, with zeros and signed
    zeros among them."""
    print("[gpu-case] split8_e2m3 records", flush=True)
    n = 64 * 32
    rng = np.random.default_rng(8)
    v = (rng.uniform(-1, 1, (n, 16)) * 2.0 ** rng.integers(-30, 1, (n, 1))).astype(np.float32)
    v[rng.uniform(size=v.shape) < 0.1] = 0.0
    v[0], v[1], v[2, :8] = 0.0, 1.0, -0.0
    v[3] = np.float32(2.0) ** -26  # below fp16: low parts only
    dev = torch.from_numpy(v).cuda()
    out = torch.zeros((n, 16), dtype=torch.int32, device="cuda")
    _run(lib.split_slices, dev.data_ptr(), out.data_ptr(), n // 64)
    got = out.cpu().numpy().view(np.uint32)
    xh = v.astype(np.float16)
    hb = xh.view(np.uint16).astype(np.uint32)
    hv = xh.astype(np.float32) * np.float32(256)
    lv = (v - xh.astype(np.float32)) * np.float32(524288)
    amax = np.maximum(np.abs(hv).max(1), np.abs(lv).max(1)).astype(np.float64)
    for t in range(n):
        # words: real parts of complex 0 1, 2 3, imaginary 0 1, 2 3, then 4 .. 7
        words = [hb[t, 4 * (j >> 2) * 2 + 4 * (j & 1) + (1 if j & 2 else 0)] |
                 (hb[t, 4 * (j >> 2) * 2 + 4 * (j & 1) + 2 + (1 if j & 2 else 0)] << 16) for j in range(8)]
        assert list(got[t, :8]) == words, t
        k = 0 if amax[t] == 0 else int(np.ceil(np.log2(amax[t] / 7.5)))
        assert amax[t] <= 7.5 * 2.0 ** k
        vals = np.concatenate([hv[t, 0::2], lv[t, 0::2], hv[t, 1::2], lv[t, 1::2]]).astype(np.float64) / 2.0 ** k
        assert list(got[t, 8:]) == _pack6(_codes(vals)) + [127 + k, 0], t
