"""The reconstruction's passes: 8 rank-one terms each, in products of 4, records newest first, then the tokens."""
import numpy as np
import pytest

from paper_2609_38166_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from oracle import oracle as O  # noqa: E402
from paper_2609_38166_amd import binding as B  # noqa: E402
from tests import gpu_harness as H  # noqa: E402

# records per tile: within a product, at the edges of products and passes, several passes
P = np.array([1, 3, 4, 5, 7, 8, 9, 15, 16, 17, 24, 25])


@pytest.mark.parametrize("gate", [synth.GATE_SCALAR, synth.GATE_DIAG])
@pytest.mark.parametrize("r,code", [(0, synth.CODE_INT8), (1, synth.CODE_INT6), (4, synth.CODE_INT4), (7, synth.CODE_INT6),
                                    (8, synth.CODE_E4M3), (9, synth.CODE_INT8), (16, synth.CODE_INT6)])
def test_partial_passes(gate, r, code):
    W, n = 25, len(P)
    wl = synth.Workload("passes", n, 1, 1, 0, W, r, gate, code=code)
    cfg, dims, rng = H.ocfg(wl), H.gdims(wl), np.random.default_rng(100 * r + 10 * code + gate)
    S = rng.standard_normal((n, 128, 128)) * (0.9 ** np.arange(128))[None, :, None]
    reps = [O.quantize(cfg, x) for x in S]
    st = B.State.empty(dims)
    H.upload_rep(st, np.arange(n), *(np.stack([getattr(x, f) for x in reps]) for f in ("Z", "delta", "c", "Kt", "Ut")))
    f16 = lambda x: x.astype(np.float16).astype(np.float64)      # noqa: E731
    a = f16(rng.uniform(0.6, 1.0, (n, W, wl.g)))
    k, u = f16(0.1 * rng.standard_normal((n, W, 128))), f16(rng.standard_normal((n, W, 128)))
    H.upload_records(st, a, k, u)
    past = torch.as_tensor(np.arange(W)[None, :] >= P[:, None], device="cuda")
    for x in (st.rec_a, st.rec_k, st.rec_u):                     # a read past the window's records would show
        x.view(n, W, -1)[past] = float("nan")
    st.rec_len.view(-1)[:] = torch.as_tensor(P, dtype=torch.int32, device="cuda")
    exp = [O.reconstruct(cfg, reps[i], None, a[i, :p], k[i, :p], u[i, :p]) for i, p in enumerate(P)]
    out = torch.empty((n, 128, 128), dtype=torch.float32, device="cuda")
    B.leapquant_dequantize_state(dims, st, out)
    got = out.cpu().numpy().transpose(0, 2, 1)
    # one rounding to fp32 (2^-24 of each entry) of sums in fp64
    assert H.rel_rows(got.reshape(n, -1), np.stack(exp).reshape(n, -1)) < 6.1e-8
    B.leapquant_window_commit(dims, st)
    rep = H.download_rep(st)
    assert np.all(rep["rec_len"] == 0) and B.leapquant_check_error(st) == 0
    want = [O.quantize(cfg, x) for x in exp]
    for f in ("Z", "delta", "c", "Kt", "Ut"):                    # decided from sums in fp64, as the oracle's
        assert np.array_equal(rep[f], np.stack([getattr(x, f) for x in want])), f


@pytest.mark.parametrize("code", [synth.CODE_INT8, synth.CODE_INT6])
@pytest.mark.parametrize("bad", [float("nan"), float("inf"), -float("inf"), None])
def test_a_residual_without_a_direction_gives_zero_pairs(bad, code):
    """A state that holds a NaN or an infinity, or only zeros (None, of either sign), has zero tokens: what remains
    is its plain quantization, and its other value channels stay finite."""
    S = torch.randn((2, 1, 128, 128), generator=torch.Generator().manual_seed(3)).cuda()     # S^T: [value][key]
    if bad is None:
        S[1] = -torch.zeros_like(S[1])
    else:
        S[1, 0, 17, 70] = bad
    st = {}
    for r in (0, 3):
        d = B.make_dims(2, 1, 1, window=4, n_comp=r, code=code)
        st[r] = B.State.empty(d)
        B.leapquant_quantize_state(d, S, st[r])
    for x in (st[3].comp_k, st[3].comp_u):
        assert x[0].view(torch.int16).any() and not x[1].view(torch.int16).any()
    for f in ("codes", "scale", "smooth"):
        a, b = (getattr(st[r], f)[1].view(torch.uint8) for r in (0, 3))
        assert torch.equal(a, b), f
    out = torch.empty_like(S)
    B.leapquant_dequantize_state(d, st[3], out)
    rest = [v for v in range(128) if v != 17]
    keys = [k for k in range(128) if k != 70]            # (an infinite row has an infinite smoothing scale)
    assert torch.isfinite(out[1, 0, rest][:, keys]).all()
