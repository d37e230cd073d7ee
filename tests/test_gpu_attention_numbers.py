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


# widths padded to 32, 64 and 128 and those that fill 32 and 128; one workgroup per problem and streamed backward
SHAPES = [(24, 6, 100), (32, 4, 100), (32, 10, 300), (40, 3, 72), (56, 6, 300), (104, 2, 100), (104, 2, 160), (128, 2, 200)]
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
@pytest.mark.parametrize("dh,heads,T", SHAPES)
def test_backward_probabilities(dh, heads, T, eps):
    """Scores of zero and row statistics of BASE and BASE + eps in turn, gradients of +1 and -1 in turn: dv sums P, dk sums dS."""
    p = block(dh, heads, T)
    unit = torch.zeros((T, dh), device="cuda")
    unit[:, 0] = 1
    sign = torch.ones((T, 1), device="cuda")
    sign[1::2] = -1
    lse = torch.full((T,), BASE, device="cuda")
    lse[1::2] += eps
    dq, dk, dv = gradients(p, unit, unit * 0, unit, unit * sign, lse)
    lo, hi = (float(t) for t in lse[:2])
    want = (T // 2) * (2.0 ** -lo - 2.0 ** -hi)
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
