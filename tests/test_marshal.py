"""The binding's native marshalling takes regular calls only; every other call goes through the Python checks."""
import pytest
import torch

from paper_2609_38166_amd import binding as B

TOKENS = ("q", "k", "v", "alpha", "beta", "o")


def _inputs(d, device):
    t = torch.ones((d.batch, d.heads_v, 128), device=device)
    k = torch.ones((d.batch, d.heads_k, 128), device=device) / 128 ** 0.5
    g = (d.batch, d.heads_v, 128) if d.gate == B.LQ_GATE_DIAG else (d.batch, d.heads_v)
    return {"q": k.clone(), "k": k, "v": t.clone(), "alpha": torch.full(g, 0.9, device=device),
            "beta": torch.full((d.batch, d.heads_v), 0.5, device=device), "o": torch.zeros_like(t)}


def test_host_tensors_are_left_to_the_python_checks():
    d = B.make_dims(2, 4, 2, window=8, n_comp=2)
    st, x = B.State.empty(d, device="cpu"), _inputs(d, "cpu")
    B.lib()
    fn = B._FN["leapquant_decode_step"]
    assert fn and B._M.step(fn, d, st, *(x[n] for n in TOKENS)) is None
    assert B._M.commit(B._FN["leapquant_window_commit"], d, st, None) is None
    assert B._M.step(fn, None, st, *(x[n] for n in TOKENS)) is None
    assert B._M.step(fn, d, object(), *(x[n] for n in TOKENS)) is None
    assert B._M.step(fn, d, st) is None
    with pytest.raises(ValueError, match="state.codes must be a device tensor"):
        B.leapquant_decode_step(d, st, *(x[n] for n in TOKENS))
    with pytest.raises(ValueError, match="device tensor"):
        B.leapquant_window_commit(d, st)
    bad = B.make_dims(2, 4, 3)
    with pytest.raises(B.LeapQuantError):
        B.leapquant_decode_step(bad, st, *(x[n] for n in TOKENS))


def _irregular(kind, d, st, x):
    """One irregular argument: what the Python checks say, or None where they take the call."""
    if kind == "dtype":
        x["q"] = x["q"].double()
        return "q must be"
    if kind == "strided":
        x["v"] = torch.ones((d.batch, d.heads_v, 256), device="cuda")[..., ::2]
        return "v must be contiguous"
    if kind == "short":
        x["o"] = x["o"][:1]
        return "o holds"
    if kind == "host":
        x["beta"] = x["beta"].cpu()
        return "beta must be a device tensor"
    if kind == "none":
        x["alpha"] = None
        return "alpha is required"
    if kind == "state":
        st.rec_u = st.rec_u[:1]
        return "state.rec_u holds"
    if kind == "address":
        x["k"] = x["k"].data_ptr()
    if kind == "subclass":
        x["k"] = torch.nn.Parameter(x["k"], requires_grad=False)
    return None


@pytest.mark.gpu
@pytest.mark.parametrize("gate", [B.LQ_GATE_SCALAR, B.LQ_GATE_DIAG])
@pytest.mark.parametrize("kind", ["regular", "dtype", "strided", "short", "host", "none", "state", "address", "subclass"])
def test_irregular_calls_do_what_the_python_path_does(kind, gate):
    d = B.make_dims(2, 4, 2, window=8, n_comp=0 if kind == "regular" else 2, gate=gate)
    got = []
    for stream in (None, torch.cuda.current_stream()):          # a given stream takes the Python path
        st, x = B.State.empty(d), _inputs(d, "cuda")
        keep = dict(x)
        B.leapquant_quantize_state(d, torch.ones((2, 4, 128, 128), device="cuda"), st)
        says = _irregular(kind, d, st, x)
        if says:
            for f in (B.leapquant_decode_step, B.leapquant_decode_step_commit):
                with pytest.raises(ValueError, match=says):
                    f(d, st, *(x[n] for n in TOKENS), stream=stream)
            assert int(st.rec_len.sum()) == 0                    # nothing was enqueued
            continue
        B.leapquant_decode_step(d, st, *(x[n] for n in TOKENS), stream=stream)
        B.leapquant_window_commit(d, st, torch.tensor([1, 0], dtype=torch.int32, device="cuda"), stream=stream)
        assert st.rec_len.view(2, 4).cpu().tolist() == [[0] * 4, [1] * 4]
        got.append([keep["o"].clone(), st.codes.clone(), st.comp_k.clone(), st.rec_u.clone()])
    for a, b in zip(*got) if got else ():
        assert torch.equal(a, b)
