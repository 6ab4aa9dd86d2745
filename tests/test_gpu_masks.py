"""Vocabulary masks that are large negative finite numbers (programs write -1e9,
-1e30 or the type's lowest value as often as -inf): in the middle and at the
end of a row, so that a lane, a segment or a wavefront's part of a row can
consist of masked columns, and at the start.  Logits need only be finite.

The references are log-sum-exps in 64 bits; a masked column adds exactly 0 to
them, so the same rows with -inf in place of the mask must also give bitwise
the same statistics."""
import pytest
import torch

import paper_2602_05774_amd as vsd
from tests.gpu_common import log

pytestmark = pytest.mark.gpu

BF, F32 = torch.bfloat16, torch.float32
# rows, columns (unmapped): the row counts and widths at which a row goes to 16, 4 and 1 wavefronts
SHAPES = {"narrow_few": (20, 9001), "narrow": (1100, 9001), "narrow_more": (1900, 9001), "wide": (20, 66001), "wide_more": (300, 66001),
          "wide_many": (2100, 66001), "one_segment": (20, 3003)}
LOWEST = "lowest"
BASE = 20   # different rows; the others repeat them
WHERE = {"middle": (0.45, 0.8), "tail": (0.5, 1.0), "last": (0.93, 1.0), "start": (0.0, 0.3)}


def _rows(V, dtype, where, mask):
    g = torch.Generator(device="cuda").manual_seed(V)
    ld = (V + 7) // 8 * 8
    lo, hi = (int(V * f) for f in WHERE[where])
    out = []
    for scale in (2.0, 3.0):
        t = torch.full((BASE, ld), 3.0e4, dtype=dtype, device="cuda")
        t[:, :V] = (scale * torch.randn(BASE, V, generator=g, device="cuda")).to(dtype)
        t[:, lo:hi] = torch.finfo(dtype).min if mask == LOWEST else mask
        out.append(t)
    live = torch.cat([torch.arange(0, lo, device="cuda"), torch.arange(hi, V, device="cuda")])
    tok = [live[torch.randint(0, live.numel(), (BASE,), generator=g, device="cuda")].to(torch.int32) for _ in range(3)]
    return out[0], out[1], tok


def _run(call, n, V, X, Y, tok, T, K):
    reps = -(-n // BASE)
    X, Y = (t.repeat(reps, 1)[:n].contiguous() for t in (X, Y))
    tok = [t.repeat(reps)[:n].contiguous() for t in tok]
    prob = vsd.Problem(1, n, 1, 1, V, V)
    params = vsd.Params(temp_draft=T, temp_target=T, kl_weight=0.3 if K else 0.0, kl_topk=K)
    if call == "score":
        sc = vsd.score_paths(prob, params, X, Y, *tok)
    elif call == "ctx":
        sc = vsd.score_paths_ctx(prob, params, [X] * 3, [Y] * 3, *tok)
    else:
        s, sc = vsd.sample_score_paths(prob, params, X, Y, None, None, 5, 1)
        tok = [s.tok_draft, s.tok_target, s.tok_greedy]
    torch.cuda.synchronize()
    assert int(sc.device_error.item()) == 0
    return sc, tok


def _check(call, shape, dtype, where, mask, T, K):
    n, V = SHAPES[shape]
    X, Y, tok = _rows(V, dtype, where, mask)
    sc, used = _run(call, n, V, X, Y, tok, T, K)
    lse = [torch.logsumexp(t[:, :V].double() / T, 1) for t in (X, Y)]
    at = torch.arange(n, device="cuda") % BASE
    # float32 sums of up to 66 001 terms of one sign, in lanes of about 1000, and results up to about 30
    for got, want in ((sc.lse_draft, lse[0]), (sc.lse_target, lse[1])):
        assert float((got.double() - want[at]).abs().max()) < 2e-5
    la = sc.log_alpha.view(n, 3).double()
    for f in range(3):
        z = used[f].long()
        d = (Y[at, z].double() - X[at, z].double()) / T - (lse[1] - lse[0])[at]
        assert float((la[:, f] - d.clamp(max=0.0)).abs().max()) < 1e-4
    inf = [t.clone() for t in (X, Y)]
    for t in inf:
        t[:, :V][t[:, :V] <= -1e8] = -float("inf")
    ref, _ = _run(call, n, V, *inf, tok, T, K)
    names = ["lse_draft", "lse_target", "log_alpha", "log_q_tok", "coef_a", "loss_pos"]
    for k in names + (["kl_idx", "kl_grad", "kl_row"] if K else []):
        assert torch.equal(getattr(sc, k), getattr(ref, k)), k


@pytest.mark.parametrize("T", (0.5, 1.0, 1.5))
@pytest.mark.parametrize("mask", (-5e9, -1e30, LOWEST), ids=str)
@pytest.mark.parametrize("call", ("score", "ctx", "one_pass"))
def test_masked_columns(call, mask, T):
    for shape in SHAPES:
        for dtype in (BF, F32):
            for where in WHERE:
                for K in (0, 5):
                    if shape == "wide_many" and where != "middle":
                        continue
                    log(f"[mask] {call} {mask} T={T} {shape} {dtype} {where} K={K}")
                    _check(call, shape, dtype, where, mask, T, K)
