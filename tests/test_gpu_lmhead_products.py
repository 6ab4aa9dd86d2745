"""The fused head's backward products at the edges of their tiles: dH = g W_d
and dW_d = g^T H_d from the g the call itself wrote (bf16), against float64
products of the same values.  Row counts, vocabularies and hidden sizes around
one 256-wide tile, K dimensions below, at and past whole 64-value stages, and
g buffers whose padding columns hold NaN (they must not be read into a
result).  Bounds: fp32 accumulation over K terms, K 2^-23 sum |a b|, and for
dH one rounding to bf16, 2^-8 |dH|.
"""
import pytest
import torch

import paper_2602_05774_amd as vsd
from tests.gpu_common import log

pytestmark = pytest.mark.gpu

DEV = "cuda"


@pytest.mark.parametrize("R,Vd", ((9, 300), (67, 40)))
def test_backward_products_of_a_wide_stride(R, Vd):
    """A gradient buffer whose row stride passes the 32-bit byte offsets of eight rows: the same as a narrow one."""
    H, ld = 128, 2 ** 28 + 64 if R < 10 else 2 ** 27 + 8
    gen = torch.Generator(device=DEV).manual_seed(R)
    rnd = lambda *s: torch.randn(*s, generator=gen, device=DEV)  # noqa: E731
    prob = vsd.Problem(1, R, 1, 1, Vd, Vd)
    head = vsd.LmHead(rnd(R, H).bfloat16(), (rnd(Vd, H) / H ** 0.5).bfloat16())
    lse = torch.logsumexp(head.hidden.double() @ head.weight.double().t(), 1).float()
    tok = [torch.randint(0, Vd, (R,), generator=gen, device=DEV, dtype=torch.int32) for _ in range(2)]
    ca, cb = rnd(R), rnd(R)
    narrow = (Vd + 7) // 8 * 8
    wide = torch.empty((R - 1) * ld + narrow, dtype=torch.bfloat16, device=DEV).as_strided((R, narrow), (ld, 1))
    res = []
    for gl in (torch.empty(R, narrow, dtype=torch.bfloat16, device=DEV), wide):
        log(f"[products] R={R} Vd={Vd} H={H} ld={gl.stride(0)}")
        grad = vsd.LmHeadGrad(torch.empty(R, H, dtype=torch.bfloat16, device=DEV), gl, torch.empty(Vd, H, device=DEV))
        res.append(vsd.weighted_loss_bwd(prob, vsd.Params(), head, lse, tok[0], tok[1], ca, cb, grad=grad))
        torch.cuda.synchronize()
    assert torch.equal(res[0].grad_logits[:, :Vd], res[1].grad_logits[:, :Vd])
    assert torch.equal(res[0].grad_hidden, res[1].grad_hidden) and torch.equal(res[0].grad_weight, res[1].grad_weight)


@pytest.mark.parametrize("T,N,L,Vd,H,pad", [
    (1, 1, 1, 40, 64, 0),       # one row, K of both products below one stage
    (17, 5, 3, 257, 192, 0),    # 255 rows; a vocabulary one past a tile
    (257, 1, 1, 64, 320, 8),    # one row past a tile; one whole stage; a wider row stride
    (64, 1, 1, 1003, 256, 0),   # whole stages of rows; an odd vocabulary
    (9, 8, 8, 512, 512, 64),    # 576 rows: everything whole
])
def test_backward_products(T, N, L, Vd, H, pad):
    gen = torch.Generator(device=DEV).manual_seed(Vd * 7 + H)
    R = T * N * L
    prob = vsd.Problem(1, T, N, L, Vd, Vd)
    rnd = lambda *s: torch.randn(*s, generator=gen, device=DEV)
    head = vsd.LmHead(rnd(R, H).bfloat16(), (rnd(Vd, H) / H ** 0.5).bfloat16())
    logits = head.hidden.double() @ head.weight.double().t()
    tok = [torch.randint(0, Vd, (R,), generator=gen, device=DEV, dtype=torch.int32) for _ in range(2)]
    ca, cb = rnd(R), rnd(R)
    ca[0], cb[0] = (0.0, 0.0) if R > 1 else (1.0, -0.5)
    ld = (Vd + 7) // 8 * 8 + pad
    gl = torch.full((R, ld), float("nan"), dtype=torch.bfloat16, device=DEV)
    grad = vsd.LmHeadGrad(torch.empty(R, H, dtype=torch.bfloat16, device=DEV), gl,
                          torch.empty(Vd, H, device=DEV))
    log(f"[products] R={R} Vd={Vd} H={H} ld={ld}")
    err = torch.zeros(1, dtype=torch.int32, device=DEV)
    vsd.weighted_loss_bwd(prob, vsd.Params(), head, torch.logsumexp(logits, 1).float(), tok[0], tok[1], ca, cb,
                          grad=grad, device_error=err)
    torch.cuda.synchronize()
    assert int(err.item()) == 0
    assert bool(torch.isnan(gl[:, Vd:].float()).all()), "padding columns were written"
    g = gl[:, :Vd].double()
    assert bool(torch.isfinite(g).all())
    rows = torch.arange(R, device=DEV)
    ref = torch.softmax(logits, 1) * (ca + cb).double()[:, None]
    ref[rows, tok[0].long()] -= ca.double()
    ref[rows, tok[1].long()] -= cb.double()
    # g: one bf16 rounding, and the float32 logit (H products) inside the exponential
    assert bool(((g - ref).abs() <= 2.0 ** -8 * ref.abs() + 1e-5 * (ca.abs() + cb.abs()).double()[:, None]).all())
    W, X = head.weight.double(), head.hidden.double()
    dh, bound = g @ W, (g.abs() @ W.abs()) * Vd * 2.0 ** -23
    assert bool(((grad.grad_hidden.double() - dh).abs() <= 2.0 ** -8 * dh.abs() + bound).all())
    dw, bound = g.t() @ X, (g.abs().t() @ X.abs()) * R * 2.0 ** -23
    assert bool(((grad.grad_weight.double() - dw).abs() <= bound + 1e-30).all())
