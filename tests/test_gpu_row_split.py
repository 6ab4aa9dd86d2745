"""A row's results do not depend on how many rows a call has: with few rows a
row is split over more wavefronts, with many it is not, and the same rows give
bitwise the same outputs either way (the many-row kernels are compared with
the oracle elsewhere).  Each case sits where the split can go wrong: fewer
chunks than wavefronts, a chunk each, remainders, a partial last chunk.
"""
import pytest
import torch

import paper_2602_05774_amd as vsd
from paper_2602_05774_amd.vsd import _query_workspace
from tests.gpu_common import log
from tests.test_gpu_parity import _custom

pytestmark = pytest.mark.gpu

BF, F32 = torch.bfloat16, torch.float32
# name: (paths of the small calls, paths of the large call, input spec)
CASES = {
    "fewer_chunks": ((1, 37), 800, dict(Vd=1003, Vt=3011, dtype=BF, mapped=True)),
    "four_chunks": ((3, 300), 800, dict(Vd=2048, Vt=2048, dtype=F32)),
    "chunk_each": ((2, 130), 800, dict(Vd=8192, Vt=8200, dtype=BF, mapped=True)),
    "remainders": ((5, 129, 600), 1200, dict(Vd=9001, Vt=20011, dtype=BF, mapped=True, map_swaps=-1)),
    "unmapped_odd": ((4, 200), 1100, dict(Vd=12345, Vt=12345, dtype=BF)),
    "ragged_f32_map": ((6, 516), 1030, dict(Vd=8709, Vt=16389, dtype=F32, mapped=True, ragged=True)),
    "masked_prefix": ((4, 130), 800, dict(Vd=9001, Vt=36000, dtype=BF, mapped=True, masked_prefix=1100)),
}
# row statistics split by the row's length too: from 4 and from 32 blocks of 2048 columns on
SCORE_CASES = dict(CASES, two_lengths=((2, 400), 600, dict(Vd=6145, Vt=65537, dtype=BF, mapped=True)),
                   wide=((1, 120, 400), 1040, dict(Vd=4099, Vt=65536, dtype=BF, mapped=True, map_swaps=-1)),
                   many_narrow=((3, 700), 4200, dict(Vd=8193, Vt=8193, dtype=BF, ragged=True)))
# one-pass draws: split by row counts of their own, and target columns past the last draft chunk's
SAMPLE_CASES = dict(CASES, long_row=((1, 384, 500), 900, dict(Vd=16389, Vt=40011, dtype=BF, mapped=True)),
                    past_the_map=((2, 200), 300, dict(Vd=4099, Vt=30000, dtype=F32, mapped=True)))
ALL_CASES = {**SCORE_CASES, **SAMPLE_CASES}
SEED, OFFSET = 77, 3


def _inputs(name):
    few, many, spec = ALL_CASES[name]
    cfg, inp = _custom(B=1, T=many, N=1, L=2, seed=sorted(ALL_CASES).index(name) + 101, **spec)
    depth = inp["valid_depth"]
    return few, many, cfg, inp["X"], inp["Y"], inp["d2t"], None if depth is None else depth.view(1, many, 1)


def _prob(cfg, n):
    return vsd.Problem(1, n, 1, 2, cfg.v_draft, cfg.v_target)


def _first(t, n, many):
    """The first n paths' part of an output of the call on all paths."""
    return t.reshape(many, -1)[:n].reshape(-1)


@pytest.mark.parametrize("name", list(CASES))
def test_sample_step(name):
    few, many, cfg, X, Y, d2t, depth = _inputs(name)

    def draw(n):
        toks = [torch.full((2 * n,), -7, dtype=torch.int32, device="cuda") for _ in range(3)]
        err = torch.zeros(1, dtype=torch.int32, device="cuda")
        for i in range(2):
            at = lambda t: t[:2 * n].view(n, 2, -1)[:, i]  # noqa: E731
            vsd.sample_step(_prob(cfg, n), i, at(X), at(Y), at(Y), d2t, None if depth is None else depth[:, :n].contiguous(),
                            0.7, 1.0, SEED, OFFSET, tokens=toks, device_error=err)
        torch.cuda.synchronize()
        assert int(err.item()) == 0
        return toks

    ref = vsd.sample_paths(_prob(cfg, many), X, Y, d2t, depth, 0.7, 1.0, SEED, OFFSET)
    ref = (ref.tok_draft, ref.tok_target, ref.tok_greedy)
    for n in few + (many,):
        log(f"[split] sample_step {name} {n} paths")
        for got, want in zip(draw(n), ref):
            assert torch.equal(got, _first(want, n, many)), n


@pytest.mark.parametrize("name", list(CASES))
def test_verify(name):
    few, many, cfg, X, Y, d2t, depth = _inputs(name)
    params = vsd.Params(temp_draft=0.7)
    smp, sc = vsd.sample_score_paths(_prob(cfg, many), params, X, Y, d2t, depth, SEED, OFFSET)

    def verify(n):
        dep = None if depth is None else depth[:, :n].contiguous()
        part = sc._replace(**{k: _first(getattr(sc, k), n, many).contiguous()
                              for k in ("log_alpha", "lse_draft", "lse_target")})
        v = vsd.verify_paths(_prob(cfg, n), params, X[:2 * n], Y[:2 * n], part, d2t, dep, SEED, OFFSET)
        torch.cuda.synchronize()
        assert int(v.device_error.item()) == 0
        return v

    ref = verify(many)
    assert int((ref.resample_tok >= 0).sum()) > 0
    for n in few:
        log(f"[split] verify {name} {n} paths")
        v = verify(n)
        assert torch.equal(v.accept_len, ref.accept_len[:n]) and torch.equal(v.resample_tok, ref.resample_tok[:n]), n


def test_verify_workspace():
    """A verification rebuilds the inverse map in the workspace and leaves every other region alone (scoring may use
    them meanwhile); the smallest workspace gives the same tokens as the one with result slots."""
    cfg, inp = _custom(B=1, T=6, N=2, L=3, Vd=2049, Vt=9000, dtype=BF, mapped=True, seed=31)
    prob, params = vsd.Problem(1, 6, 2, 3, 2049, 9000), vsd.Params()
    _, sc = vsd.sample_score_paths(prob, params, inp["X"], inp["Y"], inp["d2t"], None, SEED, OFFSET)
    need, best = _query_workspace(1, 6, 2, 3, 2049, 9000, True, 0)
    res = []
    for size in (need, best):
        log(f"[split] verify workspace {size}")
        ws = torch.full((size,), 0xA5, dtype=torch.uint8, device="cuda")
        v = vsd.verify_paths(prob, params, inp["X"], inp["Y"], sc, inp["d2t"], None, SEED, OFFSET, workspace=ws)
        torch.cuda.synchronize()
        assert int(v.device_error.item()) == 0
        written = (ws[:need] != 0xA5).nonzero().view(-1)
        assert int(written.max() - written.min()) < 4 * 9000
        assert int(written.min()) >= prob.R * 12 * 2  # past the log alpha and log q of scoring
        res.append((v.accept_len, v.resample_tok))
    assert int((res[0][1] >= 0).sum()) > 0
    assert torch.equal(res[0][0], res[1][0]) and torch.equal(res[0][1], res[1][1])


PER_ROW = ("lse_draft", "lse_target", "log_alpha", "log_q_tok", "survival", "exp_accept_len", "accept_flag",
           "valid_flag", "o_prime", "beta", "zeta", "coef_a", "coef_b", "loss_pos")
PER_ROW_KL = PER_ROW + ("kl_idx", "kl_grad", "kl_row", "kl_pos")


def _same_rows(score, few, many, K):
    ref = score(many)
    assert int(ref.device_error.item()) == 0
    for n in few:
        got = score(n)
        assert int(got.device_error.item()) == 0
        for k in PER_ROW_KL if K else PER_ROW:
            assert torch.equal(getattr(got, k).reshape(-1), _first(getattr(ref, k), n, many)), (n, k)


@pytest.mark.parametrize("K", (0, 5))
@pytest.mark.parametrize("name", list(SCORE_CASES))
def test_score(name, K):
    few, many, cfg, X, Y, d2t, depth = _inputs(name)
    params = vsd.Params(temp_draft=0.7, kl_weight=0.3 if K else 0.0, kl_topk=K)
    smp = vsd.sample_paths(_prob(cfg, many), X, Y, d2t, depth, 0.7, 1.0, SEED, OFFSET)

    def score(n):
        log(f"[split] score {name} K={K} {n} paths")
        tok = [_first(t, n, many).contiguous() for t in (smp.tok_draft, smp.tok_target, smp.tok_greedy)]
        sc = vsd.score_paths(_prob(cfg, n), params, X[:2 * n], Y[:2 * n], *tok, d2t,
                             None if depth is None else depth[:, :n].contiguous())
        torch.cuda.synchronize()
        return sc

    _same_rows(score, few, many, K)


@pytest.mark.parametrize("Vd,Vt,few,many", ((4099, 65537, (3, 257, 1000), 1030), (8193, 8193, (5, 500), 520)))
def test_score_ragged(Vd, Vt, few, many):
    """Row statistics with per-path depths at the row counts where W = 16 and W = 4 end (wide and narrow rows)."""
    g = torch.Generator(device="cuda").manual_seed(Vd)
    rnd = lambda v: (3.0 * torch.randn(2 * many, (v + 7) // 8 * 8, generator=g, device="cuda", dtype=F32)).to(BF)  # noqa: E731
    X, Y = rnd(Vd), rnd(Vt)
    d2t = None if Vd == Vt else torch.randperm(Vt, generator=g, device="cuda")[:Vd].to(torch.int32)
    tok = [torch.randint(0, Vd, (2 * many,), generator=g, device="cuda", dtype=torch.int32) for _ in range(3)]
    depth = torch.randint(1, 3, (1, many, 1), generator=g, device="cuda", dtype=torch.int32)

    def score(n):
        log(f"[split] score ragged {Vd} {Vt} {n} paths")
        sc = vsd.score_paths(vsd.Problem(1, n, 1, 2, Vd, Vt), vsd.Params(temp_draft=0.7), X[:2 * n], Y[:2 * n],
                             *[t[:2 * n] for t in tok], d2t, depth[:, :n].contiguous())
        torch.cuda.synchronize()
        return sc

    _same_rows(score, few, many, 0)


@pytest.mark.parametrize("N,L,few,many", ((1, 1, (1, 100), 2100), (7, 8, (1, 36, 40), 300), (8, 3, (5, 85, 86), 129),
                                          (9, 8, (2, 16, 17), 40), (64, 8, (1, 4, 5), 20)))
def test_combine(N, L, few, many):
    """Positions in one workgroup with the total and over many, at the edges of each."""
    cfg, inp = _custom(B=1, T=many, N=N, L=L, Vd=40, Vt=40, dtype=F32, seed=7 + N, ragged=True)
    params = vsd.Params(kl_weight=0.3, kl_topk=3)
    depth = inp["valid_depth"].view(1, many, N)

    def score(n):
        rows = n * N * L
        _, sc = vsd.sample_score_paths(vsd.Problem(1, n, N, L, 40, 40), params, inp["X"][:rows], inp["Y"][:rows], None,
                                       depth[:, :n].contiguous(), SEED, OFFSET)
        torch.cuda.synchronize()
        # at most 2100 float32 terms of a few units each, added in two orders
        assert float(sc.loss_total) == pytest.approx(float(sc.loss_pos.double().sum()), rel=1e-5, abs=1e-3)
        return sc

    _same_rows(score, few, many, 3)


@pytest.mark.parametrize("car", (vsd.VSD_CAR_PROB, vsd.VSD_CAR_LOGPROB))
@pytest.mark.parametrize("N", (1, 7, 8, 9, 40, 64))
def test_combine_kernels(N, car):
    """Paths of depth up to 8 give bitwise the same with a ninth slot that every path masks, which takes the general
    combine (a workgroup per position) instead of the small one."""
    P, V = 5, 40
    cfg, inp = _custom(B=1, T=P, N=N, L=9, Vd=V, Vt=V, dtype=F32, seed=11 + N)
    g = torch.Generator(device="cuda").manual_seed(N)
    tok = torch.randint(0, V, (3, P * N * 9), generator=g, device="cuda", dtype=torch.int32)
    depth = torch.randint(1, 9, (1, P, N), generator=g, device="cuda", dtype=torch.int32)
    params = vsd.Params(kl_weight=0.3, kl_topk=3, car_input=car)
    cut = lambda t: t.reshape(P * N, 9, -1)[:, :8].reshape(P * N * 8, -1).contiguous()  # noqa: E731
    log(f"[split] combine kernels N={N} car={car}")
    big = vsd.score_paths(vsd.Problem(1, P, N, 9, V, V), params, inp["X"], inp["Y"], *tok, None, depth)
    small = vsd.score_paths(vsd.Problem(1, P, N, 8, V, V), params, cut(inp["X"]), cut(inp["Y"]),
                            *[cut(t).view(-1) for t in tok], None, depth)
    torch.cuda.synchronize()
    assert int(big.device_error.item()) == 0 and int(small.device_error.item()) == 0
    for k in PER_ROW_KL:
        a, b = getattr(big, k), getattr(small, k)
        if k not in ("exp_accept_len", "loss_pos", "kl_pos"):
            a, b = cut(a) if a.numel() % (P * N * 9) == 0 else a, b.reshape(P * N * 8, -1)
        assert torch.equal(a, b), k


@pytest.mark.parametrize("K", (0, 5))
@pytest.mark.parametrize("name", list(SAMPLE_CASES))
def test_sample_score(name, K):
    few, many, cfg, X, Y, d2t, depth = _inputs(name)
    params = vsd.Params(temp_draft=0.7, kl_weight=0.3 if K else 0.0, kl_topk=K)
    draws = {}

    def score(n):
        log(f"[split] sample_score {name} K={K} {n} paths")
        smp, sc = vsd.sample_score_paths(_prob(cfg, n), params, X[:2 * n], Y[:2 * n], d2t,
                                         None if depth is None else depth[:, :n].contiguous(), SEED, OFFSET)
        plain = vsd.sample_paths(_prob(cfg, n), X[:2 * n], Y[:2 * n], d2t,
                                 None if depth is None else depth[:, :n].contiguous(), 0.7, 1.0, SEED, OFFSET)
        torch.cuda.synchronize()
        draws[n] = [smp.tok_draft, smp.tok_target, smp.tok_greedy]
        for a, b in zip(draws[n], (plain.tok_draft, plain.tok_target, plain.tok_greedy)):
            assert torch.equal(a, b)
        return sc

    _same_rows(score, few, many, K)
    for n in few:
        for a, b in zip(draws[n], draws[many]):
            assert torch.equal(a, _first(b, n, many)), n


@pytest.mark.parametrize("scoring", (False, True))
@pytest.mark.parametrize("Vd,Vt,H,few", ((1000, 5000, 128, (1, 96, 129)), (256, 300, 64, (3,)), (9000, 36010, 64, (5, 400)),
                                         (4097, 4097, 192, (2, 300, 768))))
def test_lm_head(Vd, Vt, H, few, scoring):
    """The fused head by single vocabulary tiles (a workspace of the best size) and by slices (the needed size, which
    has no room for the tiles' states), in runs of 1 to 6 tiles; runs of 6 cross the slices' ends."""
    many = 770
    g = torch.Generator(device="cuda").manual_seed(Vd + H)
    rnd = lambda n, std: (std * torch.randn(n, H, generator=g, device="cuda")).to(BF)  # noqa: E731
    hd, ht, wd, wt = rnd(2 * many, 1.0), rnd(2 * many, 1.0), rnd(Vd, 0.2), rnd(Vt, 0.2)
    d2t = None if Vd == Vt else torch.randperm(Vt, generator=g, device="cuda")[:Vd].to(torch.int32)
    params = vsd.Params(temp_draft=0.7)
    toks = {}

    def call(n, size):
        prob = vsd.Problem(1, n, 1, 2, Vd, Vt)
        X, Y = vsd.LmHead(hd[:2 * n].contiguous(), wd), vsd.LmHead(ht[:2 * n].contiguous(), wt)
        ws = torch.empty(size, dtype=torch.uint8, device="cuda")
        if scoring:
            tok = [torch.arange(2 * n, dtype=torch.int32, device="cuda") * k % Vd for k in (7, 11, 13)]
            sc = vsd.score_paths(prob, params, X, Y, *tok, d2t, workspace=ws)
        else:
            smp, sc = vsd.sample_score_paths(prob, params, X, Y, d2t, None, SEED, OFFSET, workspace=ws)
            tok = [smp.tok_draft, smp.tok_target, smp.tok_greedy]
        torch.cuda.synchronize()
        return tok, sc

    def score(n):
        need, best = _query_workspace(1, n, 1, 2, Vd, Vt, True, H)
        assert need < best
        log(f"[split] lm_head {Vd} {Vt} {H} scoring={scoring} {n} paths")
        toks[n], sc = call(n, best)
        tok, low = call(n, need)
        for a, b in zip(toks[n], tok):
            assert torch.equal(a, b), n
        for k in PER_ROW:
            assert torch.equal(getattr(sc, k), getattr(low, k)), (n, k)
        return sc

    _same_rows(score, few, many, 0)
    for n in few:
        for a, b in zip(toks[n], toks[many]):
            assert torch.equal(a, b[:2 * n]), n


@pytest.mark.parametrize("crowded", (False, True))
@pytest.mark.parametrize("Vd,Vt,H,paths,K", ((1000, 5000, 128, 129, 10), (256, 300, 64, 3, 16), (9000, 36010, 64, 400, 10),
                                             (4097, 4097, 192, 24, 1), (4097, 4097, 64, 768, 16)))
def test_lm_head_kl(Vd, Vt, H, paths, K, crowded):
    """The KL term's lists by runs of tiles (runs of 1 to 6, crossing the slices' ends) and by slices: the sets are exact
    either way.  crowded: the first 64 columns hold a row's best logits, so the lists cannot decide the set."""
    g = torch.Generator(device="cuda").manual_seed(Vd + H + K)
    rnd = lambda n, std: (std * torch.randn(n, H, generator=g, device="cuda")).to(BF)  # noqa: E731
    hd, ht, wd, wt = rnd(2 * paths, 1.0), rnd(2 * paths, 1.0), rnd(Vd, 0.2), rnd(Vt, 0.2)
    if crowded:
        wt[:64] *= 8
    # an ascending map that covers the first columns
    d2t = None if Vd == Vt else (torch.arange(Vd, device="cuda") * Vt // Vd).to(torch.int32)
    if d2t is not None:
        d2t[:64] = torch.arange(64, dtype=torch.int32, device="cuda")
        d2t = torch.unique(d2t)
        d2t = torch.cat([d2t, torch.tensor(sorted(set(range(Vt)) - set(d2t.tolist()))[:Vd - d2t.numel()],
                                           dtype=torch.int32, device="cuda")])
    prob = vsd.Problem(1, paths, 1, 2, Vd, Vt)
    params = vsd.Params(temp_draft=0.7, kl_weight=0.3, kl_topk=K)
    X, Y = vsd.LmHead(hd, wd), vsd.LmHead(ht, wt)
    need, best = _query_workspace(1, paths, 1, 2, Vd, Vt, True, H)
    assert need < best
    out = []
    for size in (best, need):
        log(f"[split] lm_head_kl {Vd} {Vt} {H} {paths} paths K={K} crowded={crowded} workspace {size}")
        ws = torch.empty(size, dtype=torch.uint8, device="cuda")
        smp, sc = vsd.sample_score_paths(prob, params, X, Y, d2t, None, SEED, OFFSET, workspace=ws)
        torch.cuda.synchronize()
        out.append((smp, sc))
    for a, b in zip(out[0][0], out[1][0]):
        assert torch.equal(a, b)
    for k in PER_ROW_KL:
        assert torch.equal(getattr(out[0][1], k), getattr(out[1][1], k)), k


@pytest.mark.parametrize("dtype", (BF, F32))
@pytest.mark.parametrize("V", (1, 8, 511, 512, 513, 3009, 4095, 4096))
def test_one_pass_sums_of_short_rows(V, dtype):
    """Unmapped rows of one segment (below 8 chunks of 512 columns) keep a reference per lane, the others one per row: the
    log-sum-exps against 64 bits, and with rising rows whose references move often."""
    n = 40
    g = torch.Generator(device="cuda").manual_seed(V)
    ld = (V + 7) // 8 * 8
    X, Y = (torch.full((n, ld), 3.0e4, dtype=dtype, device="cuda") for _ in range(2))
    for t, scale in ((X, 3.0), (Y, 12.0)):
        t[:, :V] = (scale * torch.randn(n, V, generator=g, device="cuda") +
                    torch.arange(V, device="cuda") * (60.0 / V) * (torch.arange(n, device="cuda") % 2)[:, None]).to(dtype)
    prob = vsd.Problem(1, n, 1, 1, V, V)
    for T in (1.0, 0.5):
        log(f"[split] short rows V={V} {dtype} T={T}")
        _, sc = vsd.sample_score_paths(prob, vsd.Params(temp_draft=T, temp_target=T), X, Y, None, None, SEED, OFFSET)
        torch.cuda.synchronize()
        for got, t in ((sc.lse_draft, X), (sc.lse_target, Y)):
            want = torch.logsumexp(t[:, :V].double() / T, 1)
            # results up to about 200, rounded to float32, and float32 sums of one sign
            assert float((got.double() - want).abs().max()) < 2e-5 * max(1.0, float(want.abs().max()) / 32)
