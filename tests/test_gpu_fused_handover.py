"""The fused step's record is read back by the commit of the same workgroup: launches of many rounds, short windows."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2609_38166_amd import binding as B  # noqa: E402


@pytest.mark.parametrize("gate", [B.LQ_GATE_SCALAR, B.LQ_GATE_DIAG])
@pytest.mark.parametrize("code,n_comp,window", [(B.LQ_CODE_INT8, 0, 1), (B.LQ_CODE_INT8, 1, 2), (B.LQ_CODE_E4M3, 0, 5),
                                                (B.LQ_CODE_BF16, 0, 3), (B.LQ_CODE_INT6, 2, 17)])
def test_every_commit_sees_its_own_last_record(code, n_comp, window, gate):
    """4096 tiles at all window positions (a scalar gate's new decay shares its line with the ones the decode has
    read): fused steps equal a decode and a commit of the full windows, byte for byte."""
    n = 4096
    d = B.make_dims(n, 1, 1, window=window, n_comp=n_comp, code=code, gate=gate)
    g = torch.Generator(device="cuda").manual_seed(window)
    rn = lambda *s: torch.randn(s, generator=g, device="cuda")      # noqa: E731
    unit = lambda x: x / x.norm(dim=-1, keepdim=True)               # noqa: E731
    fused = B.State.empty(d)
    B.leapquant_quantize_state(d, rn(n, 1, 128, 128), fused)
    fused.rec_k.copy_(0.1 * rn(*fused.rec_k.shape))
    fused.rec_u.copy_(rn(*fused.rec_u.shape))
    fused.rec_a.uniform_(0.7, 1.0, generator=g)
    fused.rec_len.copy_((torch.arange(n, device="cuda") % window).view(n, 1))
    plain = B.State(d, *[getattr(fused, f).clone() for f in B.FIELDS])
    o = [torch.empty((n, 1, 128), device="cuda") for _ in range(2)]
    for t in range(2 * window + 3):
        x = (unit(rn(n, 1, 128)), unit(rn(n, 1, 128)), rn(n, 1, 128),
             0.7 + 0.3 * torch.rand((n, 1, 128) if gate == B.LQ_GATE_DIAG else (n, 1), generator=g, device="cuda"),
             torch.rand((n, 1), generator=g, device="cuda"))
        B.leapquant_decode_step_commit(d, fused, *x, o[0])
        B.leapquant_decode_step(d, plain, *x, o[1])
        B.leapquant_window_commit(d, plain, (plain.rec_len[:, 0] == window).to(torch.int32))
        assert torch.equal(*o), t
    for f in ("codes", "scale", "smooth", "comp_k", "comp_u", "rec_len"):
        assert torch.equal(getattr(fused, f).view(torch.uint8), getattr(plain, f).view(torch.uint8)), f
    assert B.leapquant_check_error(fused) == 0 and B.leapquant_check_error(plain) == 0
