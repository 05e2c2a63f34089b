"""Linear attention at the edges of its 16-step chunks: sequences around a
chunk and a segment, every key size, decays so strong that some chunks are
taken one step at a time, and a value that is not finite, which must not reach
the outputs of the steps before it.  Against the fp64 oracle (relative L2
1e-5, the gate of every f32 path)."""
import numpy as np
import pytest
import torch

from oracle import oracle
from paper_2512_23068_amd import binding, inputs
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu

NAMES = ("q", "k", "v", "g", "dq", "dk", "dv", "dg")


def _inputs(DK, K, L, DV=64, B=1, H=2):
    cfg = inputs.LA_BY_NAME["la_tiny"].with_(batch=B, heads=H, seqlen=L, d_key=DK, d_value=DV, n_dirs=K)
    return inputs.make_la_inputs(cfg)


def _run(inp, **kw):
    d = [torch.from_numpy(np.ascontiguousarray(inp[n])).to(gu.dev()) for n in NAMES]
    out = binding.la_scan_jvp(*d, return_state=True, **kw)
    torch.cuda.synchronize()
    return out


def _check(inp, what, **kw):
    print(f"case {what}", flush=True)
    ref = oracle.la_scan_jvp(*[inp[n] for n in NAMES])
    for got, want, nm in zip(_run(inp, **kw), ref, ("o", "do", "S", "dS")):
        e = gu.rel_l2(got.cpu().numpy(), want)
        assert e <= gu.TOL, (what, nm, e)


@pytest.mark.parametrize("L", [1, 15, 16, 17, 31, 33, 130])
@pytest.mark.parametrize("DK,K", [(16, 1), (32, 2), (64, 1), (64, 2)])
def test_chunk_edges(DK, K, L):
    for seg in (0, -1, 16):
        _check(_inputs(DK, K, L), f"la chunks DK={DK} K={K} L={L} seg={seg}", seg_len=seg)


@pytest.mark.parametrize("DK,K", [(16, 2), (32, 1), (64, 1)])
def test_strong_decays(DK, K):
    """Some chunks above the exponent bound (one key, all keys, one step),
    beside ordinary ones; decays that underflow."""
    inp = _inputs(DK, K, 150, DV=128)
    g = inp["g"]
    g[:, :, 20:24, 1] = -25.0
    g[:, 0, 40:60] *= 200.0
    g[:, 1, 70] = -300.0
    inp["dg"] = np.where(np.abs(inp["dg"]) > 1, 1, inp["dg"]).astype(np.float32)
    for seg in (0, -1, 32):
        _check(inp, f"la strong decays DK={DK} K={K} seg={seg}", seg_len=seg)


@pytest.mark.parametrize("name", ["v", "dv", "k", "q"])
def test_non_finite_value_is_causal(name):
    inp = _inputs(32, 1, 64)
    ref = _run(inp, seg_len=-1)
    bad = {n: inp[n].copy() for n in NAMES}
    bad[name][..., 37, 3] = np.inf
    got = _run(bad, seg_len=-1)
    for a, b in zip(got[:2], ref[:2]):
        assert torch.allclose(a[..., :37, :], b[..., :37, :], rtol=1e-4, atol=1e-5)
    hit = got[1] if name == "dv" else got[0]
    assert not torch.isfinite(hit[..., 37, :]).all()
