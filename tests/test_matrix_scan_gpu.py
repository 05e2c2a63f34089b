"""The scan with 16 states per thread (k_scan_m) at the edges of its tiles:
fewer channels than a lane holds, channel counts around a wave's and a
block's, sequences around its four-step tiles and the segment length, rows
that are not 16-byte aligned, both input types and several states per
channel.  Against the fp64 oracle (relative L2 1e-5 per output, the gate of
every f32 path), with guard values around the outputs."""
import numpy as np
import pytest
import torch

from oracle import oracle
from paper_2512_23068_amd import binding
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu

GUARD = 64
SENTINEL = 1.25e30


def _guarded(shape):
    n = int(np.prod(shape))
    buf = torch.full((n + 2 * GUARD,), SENTINEL, device=gu.dev())
    return buf, buf[GUARD:GUARD + n].view(shape)


def _case(N, K, D, L, B=1, bf16=False, seg=0, **kw):
    what = f"N={N} K={K} D={D} L={L} B={B} bf16={bf16} seg={seg} {kw}"
    print(f"case {what}", flush=True)
    inp = gu.custom("stiff128k" if bf16 else "mamba130m", batch=B, seqlen=L, d_inner=D, d_state=N, n_dirs=K)
    if kw.get("dres"):
        inp["D_res"] = np.random.default_rng(2).standard_normal(D).astype(np.float32)
    opts = {k: kw[k] for k in ("drive", "act") if k in kw}
    x, dx = gu.inputs_to_dev(inp)
    ybuf, y = _guarded((B, L, D))
    dbuf, dy = _guarded((K, B, L, D))
    binding.scan_jvp(x, dx, gu.params_to_dev(inp), out=(y, dy), seg_len=seg, **opts)
    torch.cuda.synchronize()
    yo, dyo, _, _ = oracle.scan_jvp(inp["x"], inp["dx"], inp, **opts)
    gu.assert_close(y.cpu().numpy(), dy.cpu().numpy(), yo, dyo, what=what)
    for buf in (ybuf, dbuf):
        assert torch.all(buf[:GUARD] == SENTINEL) and torch.all(buf[-GUARD:] == SENTINEL), what


@pytest.mark.parametrize("D", [1, 2, 3, 4, 5, 7, 63, 65, 130, 255, 257])
def test_channel_edges(D):
    _case(16, 1, D, 21)
    _case(16, 2, D, 9, bf16=True)


@pytest.mark.parametrize("N,D", [(32, 1), (32, 31), (32, 33), (32, 130), (64, 1), (64, 15), (64, 17), (64, 66)])
def test_wide_states(N, D):
    _case(N, 1, D, 22)
    _case(N, 2, D, 18, bf16=True)


@pytest.mark.parametrize("L", [1, 2, 3, 4, 5, 8, 15, 16, 17, 31, 32, 33, 67])
def test_step_edges(L):
    """Segments of 16 steps: lengths around the tile and the segment."""
    _case(16, 1, 70, L, B=2, seg=16)
    _case(32, 1, 37, L, seg=-1)


@pytest.mark.parametrize("drive,act,dres", [("zoh", "identity", False), ("zoh", "silu", True), ("euler", "silu", True),
                                            ("euler", "identity", True)])
@pytest.mark.parametrize("K", [1, 2])
def test_variants_at_odd_sizes(drive, act, dres, K):
    _case(16, K, 67, 37, B=2, seg=16, drive=drive, act=act, dres=dres)


def _sequential(N, D, L, B, K=1, state=True, bf16=False, cplx=False):
    what = f"sequential N={N} D={D} L={L} B={B} K={K} bf16={bf16} complex={cplx}"
    print(f"case {what}", flush=True)
    inp = gu.custom("stiff128k" if bf16 else "mamba130m", batch=B, seqlen=L, d_inner=D, d_state=N, n_dirs=K)
    r = np.random.default_rng(5)
    h_in = dh_in = None
    if cplx:
        inp["A_im"] = r.uniform(-6.0, 6.0, (D, N)).astype(np.float32)
    if state:
        rs = lambda *s: r.standard_normal(s).astype(np.float32) + (1j * r.standard_normal(s).astype(np.float32)
                                                                   if cplx else 0)
        h_in, dh_in = rs(B, D, N), rs(K, B, D, N)
        if cplx:
            h_in, dh_in = h_in.astype(np.complex64), dh_in.astype(np.complex64)
    dev = lambda v: None if v is None else torch.from_numpy(v).to(gu.dev())
    y, dy, h, dh = gu.run(inp, h_in=dev(h_in), dh_in=dev(dh_in), return_state=True, seg_len=-1)
    yo, dyo, ho, dho = oracle.scan_jvp(inp["x"], inp["dx"], inp, h_in=h_in, dh_in=dh_in)
    gu.assert_close(y.cpu().numpy(), dy.cpu().numpy(), yo, dyo, what=what)
    for got, want, nm in ((h, ho, "h"), (dh, dho, "dh")):
        e = gu.rel_l2(got.cpu().numpy(), want)
        assert e <= gu.TOL, (what, nm, e)


@pytest.mark.parametrize("N,D", [(16, 65), (16, 66), (16, 67), (16, 257), (16, 259), (32, 33), (32, 129)])
def test_sequential_last_wave(N, D):
    """One pass whose exit state replaces its entry state, where the last wave
    has fewer channels than a lane holds: one step to five, batches of many
    waves, a host block of a single step."""
    for L in (1, 2, 5):
        _sequential(N, D, L, 300)
    _sequential(N, D, 4097, 2)
    _sequential(N, D, 7, 40, K=2, bf16=True)


@pytest.mark.parametrize("N,K,cplx", [(4, 1, False), (8, 1, False), (8, 2, False), (16, 1, True), (32, 1, True)])
def test_sequential_waves_without_channels(N, K, cplx):
    """Blocks with one wave of channels and three without, in one pass whose
    exit state replaces its entry state."""
    for D in (1, 63, 257):
        for L in (1, 2, 5):
            _sequential(N, D, L, 200, K=K, cplx=cplx)


@pytest.mark.parametrize("N,K,bf16,drive", [(16, 1, False, "euler"), (16, 2, False, "euler"), (16, 1, True, "euler"),
                                            (16, 1, False, "zoh"), (64, 2, False, "euler"), (32, 1, False, "euler")])
def test_overflow_at_the_last_step(N, K, bf16, drive):
    """After zeros a last step that overflows the state of a channel: the exit
    state is the same wherever in a tile of four steps it falls (steps past the
    sequence leave a state that is not finite as it is too)."""
    one = gu.custom("stiff128k" if bf16 else "mamba130m", batch=1, seqlen=1, d_inner=20, d_state=N, n_dirs=K)
    one["x"][:, 0, 3] = 2.0 ** 100
    one["w_delta"][3] = 1.0
    ref = None
    for L in (4, 1, 2, 3, 5, 6, 7, 8):
        inp = dict(one)
        inp["x"] = np.concatenate([np.zeros((1, L - 1, 20), np.float32), one["x"]], 1)
        inp["dx"] = np.concatenate([np.zeros((K, 1, L - 1, 20), np.float32), one["dx"]], 2)
        got = gu.run(inp, bf16=bf16, return_state=True, seg_len=-1, drive=drive)[2:]
        print(f"case overflow N={N} K={K} bf16={bf16} {drive} L={L}", flush=True)
        ref = ref or got
        assert not torch.isfinite(ref[0][:, 3]).all()
        for a, b in zip(got, ref):
            assert torch.equal(torch.isnan(a), torch.isnan(b)), L
            assert torch.equal(torch.nan_to_num(a, nan=0.0), torch.nan_to_num(b, nan=0.0)), L
