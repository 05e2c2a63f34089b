"""Linear attention at the edges of its 16-step chunks: sequences around a
chunk and a segment, every key size, strong decays and their tangents, operands
far from one, and a value that is not finite, which must not reach the outputs
of the steps before it.  Against the fp64 oracle (relative L2 1e-5, the gate of
every f32 path; where a test says so the error of the recurrence itself, a few
f32 roundings)."""
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


def _check(inp, what, tol=gu.TOL, **kw):
    print(f"case {what}", flush=True)
    ref = oracle.la_scan_jvp(*[inp[n] for n in NAMES])
    for got, want, nm in zip(_run(inp, **kw), ref, ("o", "do", "S", "dS")):
        e = gu.rel_l2(got.cpu().numpy(), want)
        print(f"  {nm} {e:.2e}", flush=True)
        assert e <= tol, (what, nm, e)


@pytest.mark.parametrize("L", [1, 15, 16, 17, 31, 33, 130])
@pytest.mark.parametrize("DK,K", [(16, 1), (32, 2), (64, 1), (64, 2)])
def test_chunk_edges(DK, K, L):
    for seg in (0, -1, 16):
        _check(_inputs(DK, K, L), f"la chunks DK={DK} K={K} L={L} seg={seg}", seg_len=seg)


@pytest.mark.parametrize("DK,K", [(16, 2), (32, 1), (64, 1)])
def test_strong_decays(DK, K):
    """One key, all keys or one step that forget nearly everything within a
    chunk (decays that underflow among them), beside ordinary ones, with the
    decays' tangents as large as the decays."""
    inp = _inputs(DK, K, 150, DV=128)
    g = inp["g"]
    g[:, :, 20:24, 1] = -25.0
    g[:, 0, 40:60] *= 200.0
    g[:, 1, 70] = -300.0
    inp["dg"] = (g * np.random.default_rng(3).standard_normal(inp["dg"].shape)).astype(np.float32)
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


# A weight is a product of at most 16 exponentials within an ulp of 6e-8 each,
# the sums over 16 steps and 64 keys round as the recurrence's do.
TIGHT = 2e-6


def _only(inp, *keep):
    """Tangents other than those named set to zero."""
    for n in ("dq", "dk", "dv", "dg"):
        if n not in keep:
            inp[n] = np.zeros_like(inp[n])
    return inp


@pytest.mark.parametrize("DK", [16, 64])
@pytest.mark.parametrize("G", [-0.5, -3.5, -12.0])
def test_operands_far_from_one(DK, G):
    """The map is linear in q, in k and in each tangent: a scale of 1e-10 or
    1e-20 changes no relative error, whatever the decay of a chunk."""
    for name in ("dq", "dk", "q", "k"):
        for scale in (1e-10, 1e-16, 1e-20, 1e10):
            inp = _inputs(DK, 1, 80)
            inp["g"] = np.full_like(inp["g"], G)
            if name.startswith("d"):
                _only(inp, name)
            inp[name] = (inp[name] * scale).astype(np.float32)
            for seg in (-1, 32):
                _check(inp, f"la scale DK={DK} g={G} {name} x {scale:g} seg={seg}", tol=TIGHT, seg_len=seg)


@pytest.mark.parametrize("DK,K", [(16, 1), (32, 2), (64, 1), (64, 2)])
@pytest.mark.parametrize("g1", [-25.0, -3.0])
def test_decay_tangent_does_not_cancel(DK, K, g1):
    """A step with a strong decay and a tangent of it of up to 3000, at every
    place of a chunk: the state before it is forgotten, so its dg hardly shows
    in the outputs after it."""
    for size in (1.0, 25.0, 300.0, 3000.0):
        inp = _inputs(DK, K, 96)
        L = inp["g"].shape[2]
        for n, t in enumerate(range(3, L, 13)):
            inp["g"][:, :, t] = g1
            inp["dg"][:, :, :, t] = size * (1 if n % 2 else -1)
        for seg in (-1, 32):
            _check(inp, f"la dg={size} DK={DK} K={K} g={g1} seg={seg}", tol=TIGHT, seg_len=seg)


def test_large_products():
    """k v in range where (q k) v is not, and the other way round."""
    for qs, ks, vs in ((1e25, 1e25, 1e-30), (1e-30, 1e-30, 1e30), (1.0, 1e20, 1e15)):
        inp = _inputs(64, 1, 40)
        for n, f in (("q", qs), ("k", ks), ("v", vs)):
            inp[n] = (inp[n] * f).astype(np.float32)
            inp["d" + n] = (inp["d" + n] * f).astype(np.float32)
        _check(inp, f"la products q {qs:g} k {ks:g} v {vs:g}", seg_len=-1)


def test_infinite_query_stays_with_its_outputs():
    """An infinite query gives infinite outputs at its step, not NaN, where it
    meets no zero."""
    inp = _inputs(32, 1, 48)
    for n in ("q", "k", "v"):
        inp[n] = np.abs(inp[n]) + 0.1
    inp["q"][:, :, 37, 3] = np.inf
    o = _run(inp, seg_len=-1)[0]
    assert torch.isposinf(o[:, :, 37]).all() and torch.isfinite(o[:, :, :37]).all()
    assert torch.isfinite(o[:, :, 38:]).all()


@pytest.mark.parametrize("K,segments", [(1, (2, 7, 8, 9, 63, 64, 65, 130)), (2, (3, 4, 5, 31, 32, 33, 70))])
def test_carry_rounds(K, segments):
    """Segments around the runs that one wave of the carry takes, and around a
    round of all its waves, with entry and exit states."""
    r = np.random.default_rng(8)
    S_in = r.standard_normal((1, 2, 16, 64)).astype(np.float32)
    dS_in = r.standard_normal((K, 1, 2, 16, 64)).astype(np.float32)
    for n in segments:
        inp = _inputs(16, K, 16 * n - 5)
        print(f"case la carry K={K} segments={n}", flush=True)
        ref = oracle.la_scan_jvp(*[inp[m] for m in NAMES], state=(S_in, dS_in))
        dev = [torch.from_numpy(v).to(gu.dev()) for v in (S_in, dS_in)]
        for got, want, nm in zip(_run(inp, seg_len=16, S_in=dev[0], dS_in=dev[1]), ref, ("o", "do", "S", "dS")):
            e = gu.rel_l2(got.cpu().numpy(), want)
            assert e <= gu.TOL, (K, n, nm, e)
