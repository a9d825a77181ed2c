"""The whole-tile kernels at the edges of arithmetic: zeros of either sign, decays that overflow FP16."""
import numpy as np
import pytest

from paper_2609_38166_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from oracle import oracle as O  # noqa: E402
from paper_2609_38166_amd import binding as B  # noqa: E402
from tests import gpu_harness as H  # noqa: E402


def _random(n, seed):
    """[n][key][value]"""
    return np.random.default_rng(seed).standard_normal((n, 128, 128)).astype(np.float32).astype(np.float64)


def _quantized(wl, S):
    dims = H.gdims(wl)
    st = B.State.empty(dims)
    B.leapquant_quantize_state(dims, H.dev(S.transpose(0, 2, 1), torch.float32), st)
    return dims, st


@pytest.mark.parametrize("code", [synth.CODE_INT8, synth.CODE_E4M3])
@pytest.mark.parametrize("kind", ["keys", "values", "sparse"])
def test_a_zero_channel_has_positive_zero_tokens(kind, code):
    """A sum of zeros of either sign is +0 (as the oracle's, which starts from 0): so are the token entries of a key
    or value channel that holds only zeros, whatever the sign of the products that meet there."""
    S = np.abs(_random(2, 4))
    if kind == "keys":                  # a zero key channel of an all-negative state
        S = -S
        S[:, [5, 77]] = 0.0
    elif kind == "values":              # a value channel of negative zeros under positive keys
        S[:, :, [5, 77]] = -0.0
    else:                               # most channels zero, their entries -0
        rng = np.random.default_rng(5)
        S = -(np.maximum(rng.standard_normal((2, 128, 1)), 0) * np.maximum(rng.standard_normal((2, 1, 128)), 0))
        S = S.astype(np.float32).astype(np.float64)
    wl = synth.Workload("zeros", 2, 1, 1, 0, 4, 1, synth.GATE_SCALAR, code=code)
    rep = H.download_rep(_quantized(wl, S)[1])
    want = [O.quantize(H.ocfg(wl), x) for x in S]
    for f in ("Kt", "Ut"):
        w = np.stack([getattr(x, f) for x in want])
        assert int((H.f16_bits(rep[f]) != H.f16_bits(w)).sum()) == 0, f
    if code == synth.CODE_E4M3:         # k~ >= 0 times +0 taken from a zero leaves it as it is
        bits = np.where(np.signbit(S), 0x80, 0)
        zero = np.broadcast_to((S == 0).all(axis=1, keepdims=True), S.shape)
        assert zero.any() or kind == "keys"
        assert int((rep["Z"][zero] != bits[zero]).sum()) == 0


# records per tile: oldest pass (and its last product of four) full or not
P = np.array([3, 4, 8, 9, 10, 14, 17, 25])


@pytest.mark.parametrize("gate", [synth.GATE_SCALAR, synth.GATE_DIAG])
def test_an_infinite_decay_meets_no_empty_slot(gate):
    """FP16 has no decay above 65504: a larger one is an infinity, which every older record and the base take over.
    The slots of a pass that hold no record take no part in it (0 times an infinity would be a NaN)."""
    n, W = len(P), 25
    wl = synth.Workload("inf", n, 1, 1, 0, W, 0, gate)
    cfg, dims, rng = H.ocfg(wl), H.gdims(wl), np.random.default_rng(8)
    reps = [O.quantize(cfg, x) for x in rng.uniform(0.5, 1.0, (n, 128, 128))]       # every code is positive
    st = B.State.empty(dims)
    H.upload_rep(st, np.arange(n), *(np.stack([getattr(x, f) for x in reps]) for f in ("Z", "delta", "c", "Kt", "Ut")))
    f16 = lambda x: x.astype(np.float16).astype(np.float64)      # noqa: E731
    a = f16(rng.uniform(0.6, 1.0, (n, W, wl.g)))
    k, u = f16(rng.uniform(0.5, 1.0, (n, W, 128))), f16(rng.uniform(0.5, 1.0, (n, W, 128)))
    a[np.arange(n), P - 1, 0] = np.inf
    H.upload_records(st, a, k, u)
    st.rec_len.view(-1)[:] = torch.as_tensor(P, dtype=torch.int32, device="cuda")
    out = torch.empty((n, 128, 128), dtype=torch.float32, device="cuda")
    B.leapquant_dequantize_state(dims, st, out)
    got = out.cpu().numpy().transpose(0, 2, 1)
    for i, p in enumerate(P):
        want = O.reconstruct(cfg, reps[i], None, a[i, :p], k[i, :p], u[i, :p])
        hit = np.zeros(128, bool)
        hit[:1 if gate else 128] = True                         # the key channels that the infinity decays
        assert np.isinf(want[hit]).mean() == 1.0 and np.isfinite(want[~hit]).all()
        assert np.isnan(got[i]).sum() == 0 and np.isinf(got[i][hit]).all(), p
        if not gate:
            continue
        # one rounding to fp32 of sums in fp64
        assert H.rel_rows(got[i][~hit].reshape(1, -1), want[~hit].reshape(1, -1)) < 6.1e-8


@pytest.mark.parametrize("gate", [synth.GATE_SCALAR, synth.GATE_DIAG])
@pytest.mark.parametrize("r,code", [(0, synth.CODE_BF16), (0, synth.CODE_E4M3), (3, synth.CODE_E4M3), (9, synth.CODE_E4M3)])
def test_a_negative_zero_stays_one(r, code, gate):
    """A sum of negative zeros is -0 in the export, and in the codes that have one (E4M3, BF16) after the commit."""
    n, W = len(P), 25
    wl = synth.Workload("mzero", n, 1, 1, 0, W, r, gate, code=code)
    cfg, dims, rng = H.ocfg(wl), H.gdims(wl), np.random.default_rng(9 + r)
    S = _random(n, 10)
    minus = rng.random(S.shape) < 0.3
    S[minus] = -0.0
    reps = [O.quantize(H.ocfg(wl, n_comp=0), x) for x in S]
    f16 = lambda x: x.astype(np.float16).astype(np.float64)      # noqa: E731
    still = np.arange(0, 128, 2)                                 # value channels that nothing is added to
    for x in reps:
        x.Kt, x.Ut = f16(rng.uniform(0, 0.1, (r, 128))), f16(rng.standard_normal((r, 128)))
        x.Ut[:, still] = -0.0
    st = B.State.empty(dims)
    H.upload_rep(st, np.arange(n), *(np.stack([getattr(x, f) for x in reps]) for f in ("Z", "delta", "c", "Kt", "Ut")))
    a = f16(rng.uniform(0.6, 1.0, (n, W, wl.g)))
    k, u = f16(rng.uniform(0, 0.1, (n, W, 128))), f16(rng.standard_normal((n, W, 128)))
    u[:, :, still] = -0.0
    H.upload_records(st, a, k, u)
    for past in (np.zeros_like(P), P):
        st.rec_len.view(-1)[:] = torch.as_tensor(past, dtype=torch.int32, device="cuda")
        want = np.stack([O.reconstruct(cfg, reps[i], None, a[i, :p], k[i, :p], u[i, :p]) for i, p in enumerate(past)])
        out = torch.empty((n, 128, 128), dtype=torch.float32, device="cuda")
        B.leapquant_dequantize_state(dims, st, out)
        got = out.cpu().numpy().transpose(0, 2, 1)
        zero = want == 0
        assert (zero & np.signbit(want) & minus).sum() > 1000 * n and np.array_equal(zero, got == 0)
        assert int((np.signbit(got) != np.signbit(want))[zero].sum()) == 0
    if r == 0:
        B.leapquant_window_commit(dims, st)
        rep = H.download_rep(st)
        assert int((rep["Z"] != np.stack([O.quantize(cfg, x).Z for x in want])).sum()) == 0


@pytest.mark.parametrize("sweeps", [1, 4, 64])
@pytest.mark.parametrize("scale", [1e-38, 1e-20, 1e-6, 1e3, 1e20, 1e36])
def test_the_sweeps_stay_in_range_at_extreme_magnitudes(scale, sweeps):
    """Sweeps are scaled by one power of two per token, taken from the largest row norm: the direction (and with it
    every token's key half) is the oracle's, which normalises every sweep, from fp32's smallest states to its largest."""
    S = _random(3, 12)
    S[1] *= 10.0 ** np.random.default_rng(13).uniform(-2, 0, (128, 1))     # rows of unlike size
    S[2] = S[2, :, :1] * S[2, :1, :]                                       # one direction, then rounding only
    S = (S * scale).astype(np.float32).astype(np.float64)
    # (a value half beyond FP16 is infinite, and what it is taken from no state: one token then)
    r = 1 if scale > 1e4 else 3
    wl = synth.Workload("extreme", 3, 1, 1, 0, 4, r, synth.GATE_SCALAR)
    cfg = H.ocfg(wl, power_iters=sweeps)
    dims = H.gdims(wl, power_iters=sweeps)
    st = B.State.empty(dims)
    B.leapquant_quantize_state(dims, H.dev(S.transpose(0, 2, 1), torch.float32), st)
    rep = H.download_rep(st)
    for i, x in enumerate(S):
        want = O.quantize(cfg, x)
        n = 1 if i == 2 else r               # past the one direction the oracle fits the rounding of its own sums
        assert np.abs(want.Kt[:n]).max() > 0
        for f in ("Kt", "Ut"):
            with np.errstate(over="ignore"):
                assert int((H.f16_bits(rep[f][i][:n]) != H.f16_bits(getattr(want, f)[:n])).sum()) == 0, (i, f)


@pytest.mark.parametrize("code", [synth.CODE_INT8, synth.CODE_BF16])
def test_a_corrupt_tile_among_others_leaves_them_alone(code):
    """An export's copies into LDS start before rec_len is known: a tile that then turns out corrupt leaves its own
    output as it was, and no copy of its behind in the LDS of the tiles that follow it on the CU."""
    n = 4096
    wl = synth.Workload("corrupt", n, 1, 1, 0, 4, 0, synth.GATE_SCALAR, code=code)
    dims = H.gdims(wl)
    st = B.State.empty(dims)
    S = torch.randn((n, 128, 128), generator=torch.Generator(device="cuda").manual_seed(7), device="cuda")
    B.leapquant_quantize_state(dims, S, st)
    whole, some = torch.empty_like(S), torch.full_like(S, 9.0)
    B.leapquant_dequantize_state(dims, st, whole)
    bad = torch.arange(n, device="cuda") % 3 != 0
    st.rec_len.view(-1)[bad] = torch.where(torch.arange(n, device="cuda") % 3 == 1, -1, 5).to(torch.int32)[bad]
    B.leapquant_dequantize_state(dims, st, some)
    assert B.leapquant_check_error(st) == B.LQ_DEVERR_BAD_REC_LEN
    assert torch.equal(some[~bad], whole[~bad]) and bool((some[bad] == 9.0).all())
