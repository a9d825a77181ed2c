"""The binding's native marshalling takes regular calls only; every other call goes through the Python checks."""
import pytest
import torch

from paper_2609_38166_amd import binding as B

TOKENS = ("q", "k", "v", "alpha", "beta", "o")
READ = ("q", "k", "b", "v", "alpha", "beta", "o")


class Tensor(torch.Tensor):
    """A tensor type of a caller's own."""


def _inputs(d, device):
    t = torch.ones((d.batch, d.heads_v, 128), device=device)
    k = torch.ones((d.batch, d.heads_k, 128), device=device) / 128 ** 0.5
    g = (d.batch, d.heads_v, 128) if d.gate == B.LQ_GATE_DIAG else (d.batch, d.heads_v)
    return {"q": k.clone(), "k": k, "b": t / 128 ** 0.5, "v": t.clone(), "alpha": torch.full(g, 0.9, device=device),
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


# kind of irregular argument: what makes it of a regular one, and what the Python checks say (None: they take it)
KINDS = {
    "dtype": (lambda t: t.double(), "must be torch.float32"),
    "strided": (lambda t: torch.stack([t, t], -1)[..., 0], "must be contiguous"),
    "short": (lambda t: t[:1], "holds"),
    "host": (lambda t: t.cpu(), "must be a device tensor"),
    "none": (lambda t: None, "is required"),
    "address": (lambda t: t.data_ptr(), None),
    "subclass": (lambda t: t.as_subclass(Tensor), None),
}


@pytest.mark.gpu
@pytest.mark.parametrize("gate", [B.LQ_GATE_SCALAR, B.LQ_GATE_DIAG])
@pytest.mark.parametrize("n_comp", [0, 2])
def test_regular_calls_take_the_native_path_and_give_the_same(n_comp, gate):
    got = {}
    for path in ("native", "python"):
        out = []
        for rule, entry, names in ((B.LQ_RULE_DELTA, "leapquant_decode_step", TOKENS),
                                   (B.LQ_RULE_DELTA, "leapquant_decode_step_commit", TOKENS),
                                   (B.LQ_RULE_GENERAL, "leapquant_decode_step_general", READ)):
            d = B.make_dims(2, 4, 2, window=8, n_comp=n_comp, gate=gate, rule=rule)
            st, x = B.State.empty(d), _inputs(d, "cuda")
            B.leapquant_quantize_state(d, torch.ones((2, 4, 128, 128), device="cuda"), st)
            mask = torch.tensor([1, 0], dtype=torch.int32, device="cuda")
            args = [x[n] for n in names]
            if path == "native":
                step = B._M.step_general if names is READ else B._M.step
                assert step(B._FN[entry], d, st, *args) == B.LQ_OK
                assert step(B._FN[entry], d, st, *args[:-1], torch.nn.Parameter(args[-1])) == B.LQ_OK   # a plain tensor too
                assert B._M.commit(B._FN["leapquant_window_commit"], d, st, mask) == B.LQ_OK
            else:
                s = torch.cuda.current_stream()          # a given stream takes the Python path
                for _ in range(2):
                    getattr(B, entry)(d, st, *args, stream=s)
                B.leapquant_window_commit(d, st, mask, stream=s)
            assert st.rec_len.view(2, 4).cpu().tolist() == [[0] * 4, [2] * 4]
            if path == "native":
                assert B._M.commit(B._FN["leapquant_window_commit"], d, st, None) == B.LQ_OK
            else:
                B.leapquant_window_commit(d, st, stream=s)
            assert int(st.rec_len.sum()) == 0
            out += [x["o"].clone(), st.codes.clone(), st.scale.clone(), st.comp_k.clone(), st.comp_u.clone(),
                    st.rec_u.clone(), st.rec_a.clone()]
        got[path] = out
    for a, b in zip(got["native"], got["python"]):
        assert torch.equal(a, b)


@pytest.mark.gpu
@pytest.mark.parametrize("kind", list(KINDS))
@pytest.mark.parametrize("name", READ)
def test_an_irregular_token_is_left_to_the_python_checks(name, kind):
    make, says = KINDS[kind]
    for entry, names, rule in (("leapquant_decode_step", TOKENS, B.LQ_RULE_DELTA),
                               ("leapquant_decode_step_commit", TOKENS, B.LQ_RULE_DELTA),
                               ("leapquant_decode_step_general", READ, B.LQ_RULE_GENERAL)):
        if name not in names:
            continue
        d = B.make_dims(2, 4, 2, window=8, n_comp=2, gate=B.LQ_GATE_DIAG, rule=rule)
        st, x = B.State.empty(d), _inputs(d, "cuda")
        kept = dict(x, **{name: make(x[name])})
        args = [kept[n] for n in names]
        native = B._M.step_general if names is READ else B._M.step
        assert native(B._FN[entry], d, st, *args) is None
        assert int(st.rec_len.sum()) == 0                        # nothing was enqueued
        if says:
            with pytest.raises(ValueError, match=f"{name} {says}"):
                getattr(B, entry)(d, st, *args)
            assert int(st.rec_len.sum()) == 0
        else:
            getattr(B, entry)(d, st, *args)
            assert int(st.rec_len.sum()) == 2 * 4


@pytest.mark.gpu
@pytest.mark.parametrize("kind", list(KINDS))
def test_an_irregular_state_or_mask_is_left_to_the_python_checks(kind):
    make, says = KINDS[kind]
    d = B.make_dims(2, 4, 2, window=8, n_comp=2)
    for field in ("rec_u", "comp_k", "rec_len"):
        if kind == "dtype":
            continue                                             # (the state's types are the caller's)
        st, x = B.State.empty(d), _inputs(d, "cuda")
        whole = st.rec_len
        setattr(st, field, make(getattr(st, field)))
        args = [x[n] for n in TOKENS]
        assert B._M.step(B._FN["leapquant_decode_step"], d, st, *args) is None
        assert B._M.commit(B._FN["leapquant_window_commit"], d, st, None) is None
        if says:
            for call in (lambda: B.leapquant_decode_step(d, st, *args), lambda: B.leapquant_window_commit(d, st)):
                with pytest.raises(ValueError, match=f"state.{field} {says}"):
                    call()
        assert int(whole.sum()) == 0
    st, x = B.State.empty(d), _inputs(d, "cuda")
    B.leapquant_quantize_state(d, torch.ones((2, 4, 128, 128), device="cuda"), st)
    B.leapquant_decode_step(d, st, *(x[n] for n in TOKENS))
    if kind in ("dtype", "none"):
        return                                                   # (a mask of any 4-byte type, or none, is regular)
    mask = make(torch.tensor([1, 0], dtype=torch.int32, device="cuda"))
    assert B._M.commit(B._FN["leapquant_window_commit"], d, st, mask) is None
    assert int(st.rec_len.sum()) == 8
    if says:
        with pytest.raises(ValueError, match=f"mask {says}"):
            B.leapquant_window_commit(d, st, mask)
        assert int(st.rec_len.sum()) == 8
    else:
        B.leapquant_window_commit(d, st, mask)
        assert int(st.rec_len.sum()) == 4
