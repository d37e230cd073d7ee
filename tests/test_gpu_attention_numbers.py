"""Attention on the matrix cores for head widths other than 64 holds probabilities and dS in 32 bits: sums whose terms cancel down to
what a shorter mantissa would lose, through the public calls, on one attention sub-block of a transformer stack."""
import numpy as np
import pytest
import torch

from paper_2501_17086_amd import binding as B
from paper_2501_17086_amd import synth

pytestmark = pytest.mark.gpu


def block(dh, heads, T, seqs=1, causal=False):
    """A Problem of one attention sub-block and one MLP sub-block whose weights are zero; Wo is the identity, Wqkv zero."""
    d = dh * heads
    w = synth.scaled(synth.WORKLOADS["gpt2_paper"], name=f"attn_{dh}_{heads}_{T}", L=2, N=seqs * T, seq_len=T, d=d, heads=heads, d_ff=8,
                     norm="none", causal=causal, gamma=0.0)
    z = lambda *s: np.zeros(s, np.float32)
    inp = {"W1": z(1, 8, d), "W2": z(1, d, 8), "U": None, "Wqkv": z(1, 3 * d, d), "Wo": np.eye(d, dtype=np.float32)[None],
           "x0": z(seqs * T, d), "e": z(seqs * T, d), "lam": None, "xin": None}
    return B.allocate(w, inp)


# widths padded to 32, 64 and 128 and those that fill 32 and 128; one workgroup per problem and streamed backward.  These are few problems:
# from four tiles of 32 positions on, a workgroup's wavefronts share one tile's keys (queries) out.
SHAPES = [(24, 6, 100), (32, 4, 100), (32, 10, 300), (40, 3, 72), (56, 6, 300), (104, 2, 100), (104, 2, 160), (128, 2, 200)]
# many (more than 256 tiles, 512 at widths to 32): a tile per wavefront, streamed both ways
SHAPES += [(24, 52, 290), (32, 52, 290), (40, 26, 300), (56, 26, 290), (104, 26, 290), (128, 26, 290)]
EPS = [1.37 * 2.0 ** -14, 1.83 * 2.0 ** -14]
BASE = 0.45           # the probabilities are 2^-BASE and (1 - eps) times that: no short numbers
# a bf16 result (2^-9) of terms that are each within 2^-23 of their value, 2e-3 of eps; 16 bits of mantissa are up to 6e-2 of it off
TOL = 2.0 ** -9 + 2e-3


def bf(v):
    return float(torch.tensor(v).bfloat16())


@pytest.mark.parametrize("eps", EPS)
@pytest.mark.parametrize("dh,heads,T", SHAPES)
def test_forward_probabilities(dh, heads, T, eps):
    """Equal queries; keys whose probabilities are p and p (1 - eps) in turn, values +1 and -1 in turn, and one key above them."""
    p = block(dh, heads, T)
    d = dh * heads
    a = np.array([bf(BASE * np.log(2) * np.sqrt(dh)), 0, 0, bf(-eps * np.sqrt(dh))])      # the first key, the second, p, p (1 - eps)
    p.x[0, :, 0] = 1
    p.x[0, 3::2, 1], p.x[0, 0, 1] = a[3], a[0]
    p.x[0, 2::2, 2], p.x[0, 3::2, 2] = 1, -1
    for h in range(heads):
        p.Wqkv[0, h * dh, 0] = 1
        p.Wqkv[0, d + h * dh, 1] = 1
        p.Wqkv[0, 2 * d + h * dh + dh - 1, 2] = 1
    B.hbp_forward(p)
    s = np.exp(a / np.sqrt(dh))
    n = T // 2 - 1
    want = n * (s[2] - s[3]) / (s[0] + s[1] + n * (s[2] + s[3]))
    got = p.attn_o[0].float().reshape(T, heads, dh)[..., -1].cpu().numpy()
    assert np.abs(got / want - 1).max() < TOL, (got.min() / want - 1, got.max() / want - 1)


def gradients(p, q, k, v, do, lse):
    """dq, dk, dv [T, heads, dh] by way of the gradient of Wqkv: the block's input is the identity matrix."""
    T, d = p.x.shape[1], p.x.shape[2]
    heads = p.desc.heads
    p.x[0].copy_(torch.eye(d, device="cuda")[:T])
    p.qkv[0].copy_(torch.cat([t.repeat(1, heads) for t in (q, k, v)], 1))
    p.g[1].copy_(do.repeat(1, heads))
    p.lse[0].reshape(heads, T).copy_(lse.expand(heads, T))
    p.attn_o.zero_()
    B.hbp_param_grads(p)
    return [t[:, :T].reshape(heads, -1, T).permute(2, 0, 1).cpu().numpy() for t in p.dWqkv[0].chunk(3)]


@pytest.mark.parametrize("eps", EPS)
@pytest.mark.parametrize("score", [0, 13])
@pytest.mark.parametrize("dh,heads,T", SHAPES)
def test_backward_probabilities(dh, heads, T, score, eps):
    """Equal scores (in base 2) and row statistics BASE and BASE + eps above them in turn, gradients of +1 and -1 in turn: dv sums P,
    dk sums dS."""
    p = block(dh, heads, T)
    unit = torch.zeros((T, dh), device="cuda")
    unit[:, 0] = 1
    sign = torch.ones((T, 1), device="cuda")
    sign[1::2] = -1
    k = unit * bf(score * np.log(2) * np.sqrt(dh))
    t = float(k[0, 0]) / np.sqrt(dh) / np.log(2)
    lse = torch.full((T,), t + BASE, device="cuda")
    lse[1::2] += eps
    dq, dk, dv = gradients(p, unit, k, unit, unit * sign, lse)
    lo, hi = (float(x) for x in lse[:2])
    want = (T // 2) * (2.0 ** (t - lo) - 2.0 ** (t - hi))
    assert np.abs(dv[..., 0] / want - 1).max() < TOL, np.abs(dv[..., 0] / want - 1).max()
    assert np.abs(dk[..., 0] / (want / np.sqrt(dh)) - 1).max() < TOL, np.abs(dk[..., 0] / (want / np.sqrt(dh)) - 1).max()


@pytest.mark.parametrize("eps", EPS)
@pytest.mark.parametrize("dh,heads,T", SHAPES)
def test_backward_score_gradients(dh, heads, T, eps):
    """dS of p and -p (1 - eps) in turn along a row: dq sums them."""
    p = block(dh, heads, T)
    unit = torch.zeros((T, dh), device="cuda")
    unit[:, 0] = 1
    v, do = unit.clone(), unit.clone()
    v[1::2, 0], v[1::2, 1], do[:, 1] = -1, eps, 1
    dq, dk, dv = gradients(p, unit * 0, unit, v, do, torch.full((T,), BASE, device="cuda"))
    want = (T // 2) * 2.0 ** -BASE * bf(eps) / np.sqrt(dh)
    assert np.abs(dq[..., 0] / want - 1).max() < TOL, np.abs(dq[..., 0] / want - 1).max()


# ---- infinities and NaNs reach what sees them, and nothing else: not what the mask, the sequence's end or a padded width leaves out ----
WIDE = [(24, 2, 72), (32, 2, 100), (32, 2, 260), (40, 2, 40), (56, 2, 270), (104, 2, 100), (104, 2, 150), (128, 2, 130)]
WIDE += [(24, 29, 270), (32, 29, 270), (56, 29, 270), (104, 29, 270), (128, 29, 270)]       # (many problems, as above: 522 tiles)


def checked(heads):
    """The heads that are compared: of many, the first, whose numbers are planted, the second and the last."""
    return range(heads) if heads <= 2 else (0, 1, heads - 1)


def heads_of(t, seqs, T, heads, parts):
    """[N, parts d] -> parts x [seqs, heads, T, dh], float64"""
    return np.moveaxis(t.double().cpu().numpy().reshape(seqs, T, parts, heads, -1), (2, 3), (0, 2))


def visible(causal, i, T):
    return slice(0, i + 1 if causal else T)


def plain_forward(q, k, v, causal):
    T, dh = q.shape
    o, lse = np.empty_like(q), np.empty(T)
    for i in range(T):
        sl = visible(causal, i, T)
        s = (k[sl] @ q[i]) / np.sqrt(dh)
        m = np.fmax.reduce(s)
        pr = np.exp(s - m)
        o[i] = (pr[:, None] * v[sl]).sum(0) / pr.sum()
        lse[i] = (m + np.log(pr.sum())) / np.log(2)
    return o, lse


def finite_forward(q, k, v, causal):
    """The same for all heads [sequences, heads, T, dh] of finite data."""
    T, dh = q.shape[-2:]
    s = q @ np.swapaxes(k, -1, -2) / np.sqrt(dh)
    if causal:
        s = np.where(np.tril(np.ones((T, T), bool)), s, -np.inf)
    lse = np.logaddexp.reduce(s, axis=-1)
    return np.exp(s - lse[..., None]) @ v, lse / np.log(2)


def plain_backward(q, k, v, do, o, lse, causal):
    T, dh = q.shape
    dq, dk, dv = np.zeros_like(q), np.zeros_like(q), np.zeros_like(q)
    for i in range(T):
        sl = visible(causal, i, T)
        pr = np.exp2((k[sl] @ q[i]) / np.sqrt(dh) / np.log(2) - lse[i])
        ds = pr * (v[sl] @ do[i] - (do[i] * o[i]).sum())
        dq[i] = (ds[:, None] * k[sl]).sum(0) / np.sqrt(dh)
        dk[sl] += ds[:, None] * q[i] / np.sqrt(dh)
        dv[sl] += pr[:, None] * do[i]
    return dq, dk, dv


def assert_same(got, want, what):
    assert np.array_equal(np.isnan(got), np.isnan(want)), f"{what}: NaN"
    inf = np.isinf(want)
    assert np.array_equal(np.isinf(got), inf) and np.array_equal(got[inf], want[inf]), f"{what}: infinities"
    m = np.isfinite(want)
    assert np.linalg.norm(got[m] - want[m]) <= 1e-2 * np.linalg.norm(want[m]) + 1e-30, what


@pytest.mark.parametrize("plant", ["nan", "inf_value", "inf_key"])
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("dh,heads,T", WIDE)
def test_forward_with_infinities(dh, heads, T, causal, plant):
    S, d = 2, dh * heads
    p = block(dh, heads, T, seqs=S, causal=causal)
    gen = torch.Generator(device="cuda").manual_seed(1)
    p.x[0] = torch.randn((S * T, d), generator=gen, device="cuda")
    p.Wqkv[0] = torch.randn((3 * d, d), generator=gen, device="cuda") * (0.7 / np.sqrt(d))
    # column 0 of the input overflows one column of one head: the last one, of the values or of the keys
    p.x[0, :, 0] = 0
    p.Wqkv[0, :, 0] = 0
    last = dh - 1                                  # (of the first head)
    if plant == "inf_key":                         # minus infinity against a positive query: a probability of zero
        p.Wqkv[0, last] = 0
        p.x[0, :, 1] = 1
        p.Wqkv[0, :, 1] = 0
        p.Wqkv[0, last, 1] = 1
    p.Wqkv[0, (2 * d if plant == "inf_value" else d) + last, 0] = -100
    t = T - 3
    if plant == "nan":
        p.x[0, t] = float("nan")
    else:
        p.x[0, t, 0] = 2e38
    B.hbp_forward(p)
    q, k, v = heads_of(p.qkv[0], S, T, heads, 3)
    assert not np.isfinite(k if plant == "inf_key" else v).all()
    got = heads_of(p.attn_o[0], S, T, heads, 1)[0]
    lse = p.lse[0].double().cpu().numpy().reshape(S, heads, T)
    with np.errstate(invalid="ignore"):
        for s in range(S):
            for h in checked(heads):
                o, L = plain_forward(q[s, h], k[s, h], v[s, h], causal)
                assert_same(got[s, h], o, f"o, sequence {s}, head {h}")
                assert_same(lse[s, h], L, f"lse, sequence {s}, head {h}")


@pytest.mark.parametrize("plant", ["nan_value", "inf_value", "inf_key", "inf_query", "nan_gradient"])
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("dh,heads,T", WIDE)
def test_backward_with_infinities(dh, heads, T, causal, plant):
    """By token: the product with Wqkv carries what is not finite to all columns of its row."""
    S, d = 2, dh * heads
    p = block(dh, heads, T, seqs=S, causal=causal)
    gen = torch.Generator(device="cuda").manual_seed(2)
    p.Wqkv[0] = torch.eye(d, device="cuda").repeat(3, 1)
    qkv = torch.randn((S * T, 3 * d), generator=gen, device="cuda").bfloat16()
    qkv[:, dh - 1] = qkv[:, dh - 1].abs() + 0.25
    do = torch.randn((S * T, d), generator=gen, device="cuda").bfloat16()
    q, k, v = heads_of(qkv, S, T, heads, 3)
    o, lse = finite_forward(q, k, v, causal)
    p.attn_o[0] = torch.from_numpy(o).permute(0, 2, 1, 3).reshape(S * T, d).to("cuda")
    p.lse[0] = torch.from_numpy(lse.reshape(-1)).to("cuda")
    t = T - 3
    col = {"inf_value": 2 * d, "inf_key": d, "inf_query": 0}
    if plant == "nan_value":
        qkv[t, 2 * d:] = float("nan")
    elif plant == "nan_gradient":
        do[t] = float("nan")
    else:
        qkv[t, col[plant] + dh - 1] = -float("inf")
    p.qkv[0], p.e[:] = qkv, do
    B.hbp_exact_backward(p)
    q, k, v = heads_of(qkv, S, T, heads, 3)
    g, oo = heads_of(do, S, T, heads, 1)[0], heads_of(p.attn_o[0], S, T, heads, 1)[0]
    lse = p.lse[0].double().cpu().numpy().reshape(S, heads, T)
    hs = list(checked(heads))
    want = np.zeros((S, len(hs), T, dh))
    with np.errstate(invalid="ignore"):
        for s in range(S):
            for i, h in enumerate(hs):
                want[s, i] = g[s, h] + sum(plain_backward(q[s, h], k[s, h], v[s, h], g[s, h], oo[s, h], lse[s, h], causal))
    want = want.transpose(0, 2, 1, 3).reshape(S * T, -1)
    got = p.g[0].double().cpu().numpy().reshape(S * T, heads, dh)[:, hs].reshape(S * T, -1)
    bad = ~np.isfinite(want).all(1)
    assert np.array_equal(~np.isfinite(got).all(1), bad), (np.flatnonzero(bad), np.flatnonzero(~np.isfinite(got).all(1)))
    assert np.linalg.norm(got[~bad] - want[~bad]) <= 1e-2 * np.linalg.norm(want[~bad]) + 1e-30


# ---- keys whose scores are all minus infinity weigh nothing, whichever of a wavefront's tiles they fill ----
# few problems (a workgroup's wavefronts share one tile's keys out: key tiles 0 to 3 are each one's first) and many (a tile each)
@pytest.mark.parametrize("plant", ["inf_key", "overflow"])
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("dh,heads,T,tile", [(64, 2, 200, t) for t in range(7)] + [(64, 52, 320, 0), (64, 52, 320, 3), (24, 2, 130, 0),
                                                                                  (32, 2, 130, 2), (56, 2, 200, 1), (128, 2, 200, 3)])
def test_forward_with_hidden_keys(dh, heads, T, tile, causal, plant):
    d = dh * heads
    p = block(dh, heads, T, causal=causal)
    gen = torch.Generator(device="cuda").manual_seed(3)
    x = torch.randn((T, d), generator=gen, device="cuda")
    wqkv = torch.randn((3 * d, d), generator=gen, device="cuda") * (0.7 / np.sqrt(d))
    # the last column of every head: a positive query, and from column 0 of the input a key of minus infinity, or a finite one whose
    # product with the query is
    hidden = slice(32 * tile, min(32 * tile + 32, T))
    x[:, 0], x[:, 1] = 0, 1
    x[hidden, 0] = 2e38
    wqkv[:, :2] = 0
    last = torch.arange(heads, device="cuda") * dh + dh - 1
    wqkv[last] = 0
    wqkv[last, 1] = 16
    wqkv[d + last, 0] = -100 if plant == "inf_key" else -1
    p.x[0], p.Wqkv[0] = x, wqkv
    B.hbp_forward(p)
    q, k, v = heads_of(p.qkv[0], 1, T, heads, 3)
    assert np.isinf(k[0, :, hidden, -1]).all() if plant == "inf_key" else np.isfinite(k).all()
    k[0, :, hidden, -1] = -np.inf
    got = heads_of(p.attn_o[0], 1, T, heads, 1)[0]
    lse = p.lse[0].double().cpu().numpy().reshape(1, heads, T)
    with np.errstate(invalid="ignore"):
        for h in {0, 1, heads - 1}:
            o, L = plain_forward(q[0, h], k[0, h], v[0, h], causal)
            assert np.isfinite(L).sum() == (T - 32 if causal and tile == 0 else T)      # (the others see hidden keys only)
            assert_same(got[0, h], o, f"o, head {h}")
            assert_same(lse[0, h], L, f"lse, head {h}")
