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
