"""What a program that uses this framework has it compute, as measured cases.

Every case is one pass through the binding's entry points on a stack of residual blocks:

  grad     hbp_backward(k) and hbp_param_grads on a saved forward state      (the Highway-BP step itself)
  exact    hbp_exact_backward and hbp_param_grads on a saved forward state   (the comparison the paper draws)
  forward  hbp_forward                                                       (what fills the saved state)
  both     hbp_forward, hbp_backward(k), hbp_param_grads                     (a program with its own loss)
  train    hbp_train_step: forward, loss, backward, parameter gradients, AdamW

The saved state of "grad" and "exact" is made by plain torch in the storage precision, so that what is measured
does not depend on the forward pass.  Sizes are those of synth.WORKLOADS, cut in depth or tokens where a full stack
would not fit three times on a card, and generic odd ones beside them.
"""
import math

import torch

from paper_2501_17086_amd import binding as B

CELLS = ("gated", "lstm", "gru")
RECURRENT = ("rnn",) + CELLS
EPS = 1e-6

_MLP = dict(kind="mlp", dtype="bf16", act="gelu", norm="rms", lam="uniform", lam_lo=0.9, post="none", gamma=0.0,
            w_std=0.0, k=2, every=False)
_TFM = dict(kind="transformer", dtype="bf16", act="gelu", norm="rms", lam="one", lam_lo=1.0, post="none", gamma=0.2,
            w_std=0.02, k=2, every=False)
_REC = dict(dtype="bf16", act="tanh", norm="none", lam="sigmoid", lam_lo=0.0, post="none", gamma=0.0, w_std=0.0, k=2,
            every=True)
_GATES = {"gated": 2, "lstm": 2, "gru": 3}     # d_ff / d of the cells


def listed():
    return [
        # the small fp32 stack (8 blocks, 128 tokens): a reference-precision check run, launches and latency
        dict(_MLP, name="mlp_f32_small", op="grad", dtype="f32", norm="none", lam="one", L=8, N=128, d=64, d_ff=256),
        # a small bf16 stack at sizes that fit no tile: fine-tuning on one odd batch, forward and backward
        dict(_MLP, name="mlp_odd", op="both", L=12, N=1000, d=328, d_ff=1304),
        # the paper's residual-network depth at full size, the backward pass of one training step
        dict(_MLP, name="mlp_resnet_grad", op="grad", L=32, N=8192, d=512, d_ff=2048),
        # the same stack's exact backpropagation, block after block
        dict(_MLP, name="mlp_resnet_exact", op="exact", L=32, N=8192, d=512, d_ff=2048),
        # transformer widths, forward only: 6 of 48 blocks
        dict(_MLP, name="mlp_wide_forward", op="forward", lam="one", w_std=0.02, L=6, N=16384, d=1024, d_ff=4096),
        # the widest stack, 8 of 96 blocks: the largest products
        dict(_MLP, name="mlp_large_grad", op="grad", lam_lo=0.8, w_std=0.02, L=8, N=16384, d=2048, d_ff=8192),
        # the paper's GPT-2 configuration (12 layers of width 256, 128 sequences of 256): a whole training step
        dict(_TFM, name="tfm_gpt2_train", op="train", L=24, N=128 * 256, d=256, d_ff=1024, heads=4, seq_len=256,
             causal=True),
        # longer sequences, wider layers: 3 of 12 layers, 16 sequences of 1024, where attention weighs most
        dict(_TFM, name="tfm_long_grad", op="grad", L=6, N=16 * 1024, d=1024, d_ff=4096, heads=16, seq_len=1024,
             causal=True),
        # a small transformer with narrow heads and ragged sequences, not causal, post-norm layers (the paper's
        # RoBERTa paragraph), forward and backward
        dict(_TFM, name="tfm_small_post", op="both", norm="none", post="rms", gamma=0.8, L=8, N=12 * 100, d=256,
             d_ff=1024, heads=8, seq_len=100, causal=False),
        # the recurrent stack along time (4096 steps, batch 32, contractive weights): the Highway-BP step
        dict(_REC, name="rnn_grad", op="grad", kind="rnn", L=4096, N=32, d=1024, d_ff=1024, d_in=1024),
        # its forward pass step by step and exact backpropagation through time are what a program without the
        # iteration runs; a quarter of the steps
        dict(_REC, name="rnn_exact", op="exact", kind="rnn", L=1024, N=32, d=1024, d_ff=1024, d_in=1024),
        # the standard GRU, the cell of the paper's recurrent experiments: forward and backward of a training step
        dict(_REC, name="gru_both", op="both", kind="gru", L=1024, N=32, d=1024, d_ff=3072, d_in=1024),
    ]


def _log(rng, lo, hi, step):
    """A multiple of `step` between lo and hi, spread over the logarithm."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(lo, min(hi, int(round(v / step)) * step))


def draw(rng):
    fam = rng.choice(("f32", "mlp", "mlp", "tfm", "tfm", "rnn", "cell"))
    if fam == "f32":
        d = _log(rng, 32, 256, 8)
        return dict(_MLP, op=rng.choice(("grad", "both", "exact")), dtype="f32", norm=rng.choice(("none", "rms")),
                    lam=rng.choice(("one", "uniform")), L=rng.randint(3, 12), N=_log(rng, 32, 1024, 1), d=d,
                    d_ff=d * rng.choice((2, 4)), k=rng.randint(0, 3))
    if fam == "mlp":
        d = _log(rng, 64, 1536, 8) if rng.random() < 0.5 else 64 * _log(rng, 1, 24, 1)
        cap = 2.0e9 / (d * d)                      # tokens x blocks: the cost of a case stays bounded
        N = _log(rng, 16, max(64, int(min(16384, cap / 4))), 1)
        if rng.random() < 0.5 and N > 256:
            N = N // 128 * 128
        post = rng.choice(("none", "none", "rms"))
        return dict(_MLP, op=rng.choice(("grad", "grad", "both", "forward", "exact")), L=rng.randint(4, 24), N=N, d=d,
                    d_ff=d * rng.choice((2, 4)), lam=rng.choice(("one", "uniform")), post=post,
                    norm="rms" if post == "none" else "none", gamma=0.0 if post == "none" else 0.8, k=rng.randint(0, 3))
    if fam == "tfm":
        dh = rng.choice((32, 64, 64, 128))
        heads = rng.choice((2, 4, 8, 12))
        T = _log(rng, 16, 1024, 1) if rng.random() < 0.5 else rng.choice((64, 128, 256, 512, 1024))
        d = dh * heads
        seqs = max(1, _log(rng, 1, 64 if dh == 64 else 16, 1) * 256 // max(T, 64))
        return dict(_TFM, op=rng.choice(("grad", "both", "train")), L=2 * rng.randint(1, 6), N=seqs * T, d=d, d_ff=4 * d,
                    heads=heads, seq_len=T, causal=rng.random() < 0.6, gamma=rng.choice((0.0, 0.2)),
                    k=rng.randint(1, 3))
    kind = "rnn" if fam == "rnn" else rng.choice(CELLS)
    H = 64 * _log(rng, 2, 16, 1) if rng.random() < 0.7 else _log(rng, 104, 1000, 8)
    d = 2 * H if kind == "lstm" else H
    return dict(_REC, op=rng.choice(("grad", "both", "exact", "forward")), kind=kind, L=_log(rng, 64, 1024, 1),
                N=rng.choice((1, 8, 20, 32, 32, 64)), d=d, d_ff=d if kind == "rnn" else d * _GATES[kind],
                d_in=H, k=rng.randint(1, 3))


# ---------------------------------------------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------------------------------------------
def _storage(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _weight_shapes(case):
    L, d, F = case["L"], case["d"], case["d_ff"]
    kind = case["kind"]
    if kind == "mlp":
        return {"W1": (L, F, d), "W2": (L, d, F)}
    if kind == "transformer":
        n = L // 2
        return {"W1": (n, F, d), "W2": (n, d, F), "Wqkv": (n, 3 * d, d), "Wo": (n, d, d)}
    if kind == "rnn":
        return {"W1": (F, d), "W2": (d, F), "U": (F, case["d_in"])}
    return {"W1": (F, d // 2 if kind == "lstm" else d), "U": (F, case["d_in"])}


def _inputs(case, seed):
    """Weights, stack input, coefficients and loss gradient (or target) in the storage type, from the seed alone."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    dt = _storage(case)
    L, N, d, F, kind = case["L"], case["N"], case["d"], case["d_ff"], case["kind"]

    def normal(shape, std=1.0):
        return torch.randn(shape, generator=gen, device="cuda").mul_(std).to(dt)

    inp = {}
    for name, shape in _weight_shapes(case).items():
        std = case["w_std"] if case["w_std"] > 0 and name != "U" else 1.0 / math.sqrt(shape[-1])
        if name in ("W2", "Wo") and case["post"] == "none" and kind in ("mlp", "transformer"):
            std /= math.sqrt(L)
        if kind == "rnn" and name != "U":
            std *= 0.25                              # contractive: exact gradients through thousands of steps stay finite
        if kind in CELLS and name == "W1":
            std *= 0.5
        inp[name] = normal(shape, std)
    if kind in RECURRENT:
        inp["x0"] = torch.zeros((N, d), dtype=dt, device="cuda")
        inp["xin"] = normal((L, N, case["d_in"]))
        if kind in CELLS:                            # the gates' constant bias comes in through input channel 0
            H = d // 2 if kind == "lstm" else d
            inp["xin"][..., 0] = 1.0
            inp["U"][:, 0] = 0.0
            if kind == "lstm":
                inp["U"][H:2 * H, 0] = 3.0
            else:
                inp["U"][:H, 0] = -3.0
    else:
        inp["x0"] = normal((N, d))
    inp["lam"] = None
    if kind not in CELLS and case["lam"] == "uniform":
        inp["lam"] = torch.rand((L, d), generator=gen, device="cuda") * (1.0 - case["lam_lo"]) + case["lam_lo"]
    elif kind not in CELLS and case["lam"] == "sigmoid":
        inp["lam"] = torch.sigmoid(torch.randn((L, d), generator=gen, device="cuda") * 0.5 + 3.0)
    if case["every"]:
        inp["e"] = normal((L + 1, N, d))
        inp["e"][0] = 0
    else:
        inp["e"] = normal((N, d))                    # (the training step's target)
    return inp


# ---------------------------------------------------------------------------------------------------------------
# the stack in plain torch: `dt` is the type computed in, values are kept in `st`
# ---------------------------------------------------------------------------------------------------------------
def _heads_view(case, t, parts):
    """[N, parts * d] -> `parts` tensors [sequences, heads, T, dh]."""
    T, h, d = case["seq_len"], case["heads"], case["d"]
    t = t.reshape(-1, T, parts, h, d // h).permute(2, 0, 3, 1, 4).contiguous()
    return [t[i] for i in range(parts)]


def _from_heads(case, parts):
    t = torch.stack(parts).permute(1, 3, 0, 2, 4).contiguous()
    return t.reshape(case["N"], -1)


def _probabilities(case, q, k):
    s = torch.matmul(q, k.transpose(-1, -2).contiguous()) / math.sqrt(q.shape[-1])
    if case["causal"]:
        T = case["seq_len"]
        s.masked_fill_(torch.ones((T, T), dtype=torch.bool, device=s.device).triu(1), float("-inf"))
    lse = torch.logsumexp(s, -1)
    return s.sub_(lse.unsqueeze(-1)).exp_(), lse * 1.4426950408889634


def _gelu(a):
    phi = 0.5 * (1.0 + torch.erf(a * 0.70710678118654752440))
    return a * phi, phi + a * torch.exp(-0.5 * a * a) * 0.39894228040143267794


def _forward(case, inp, dt, st):
    """Saved state of hbp_forward: x, y, rinv, z, dphi, lam (cells), qkv, attn_o, lse."""
    L, N, d, F, kind = case["L"], case["N"], case["d"], case["d_ff"], case["kind"]
    f32 = torch.float32 if st != torch.float64 else torch.float64
    dev = "cuda"
    tfm = kind == "transformer"
    Li = L // 2 if tfm else L
    rms, post = case["norm"] == "rms", case["post"] == "rms"
    s = {"x": torch.zeros((L + 1, N, d), dtype=st, device=dev), "z": torch.empty((Li, N, F), dtype=st, device=dev)}
    s["x"][0] = inp["x0"]
    if rms:
        s["y"] = torch.empty((L, N, d), dtype=st, device=dev)
    if rms or post:
        s["rinv"] = torch.empty((L, N), dtype=f32, device=dev)
    if case["act"] == "gelu":
        s["dphi"] = torch.empty((Li, N, F), dtype=st, device=dev)
    if tfm:
        s["qkv"] = torch.empty((Li, N, 3 * d), dtype=st, device=dev)
        s["attn_o"] = torch.empty((Li, N, d), dtype=st, device=dev)
        s["lse"] = torch.empty((Li, N * case["heads"]), dtype=f32, device=dev)
    if kind in CELLS:
        s["lam"] = torch.empty((L, N, d), dtype=st, device=dev)
    if kind in RECURRENT:
        W1 = inp["W1"].to(dt)
        W2 = inp["W2"].to(dt) if kind == "rnn" else None
        ux = torch.matmul(inp["xin"].reshape(L * N, -1).to(dt), inp["U"].to(dt).t().contiguous()).reshape(L, N, F)
        W1t = W1.t().contiguous()
        W2t = W2.t().contiguous() if W2 is not None else None
        H = d // 2 if kind == "lstm" else d
        for l in range(L):
            x = s["x"][l].to(dt)
            if kind == "rnn":
                s["z"][l] = torch.tanh(torch.addmm(ux[l], x, W1t))
                s["x"][l + 1] = torch.addmm(x * inp["lam"][l].to(dt), s["z"][l].to(dt), W2t)
            elif kind == "gated":
                p = torch.addmm(ux[l], x, W1t)
                u, c = torch.sigmoid(p[:, :H]), torch.tanh(p[:, H:])
                s["z"][l, :, :H], s["z"][l, :, H:] = u, c
                s["lam"][l] = 1.0 - u
                s["x"][l + 1] = torch.addcmul(x, u, c - x)
            elif kind == "lstm":
                p = torch.addmm(ux[l], x[:, H:], W1t)
                ifo, gg = torch.sigmoid(p[:, :3 * H]), torch.tanh(p[:, 3 * H:])
                i, f, o = ifo[:, :H], ifo[:, H:2 * H], ifo[:, 2 * H:]
                c = torch.addcmul(f * x[:, :H], i, gg)
                s["z"][l, :, :3 * H], s["z"][l, :, 3 * H:] = ifo, gg
                s["lam"][l, :, :H], s["lam"][l, :, H:] = f, 0
                s["x"][l + 1, :, :H], s["x"][l + 1, :, H:] = c, o * torch.tanh(c)
            else:
                zr = torch.sigmoid(torch.addmm(ux[l][:, :2 * H], x, W1t[:, :2 * H]))
                z, r = zr[:, :H], zr[:, H:]
                n = torch.tanh(torch.addmm(ux[l][:, 2 * H:], (r * x).to(st).to(dt), W1t[:, 2 * H:]))
                s["z"][l, :, :2 * H], s["z"][l, :, 2 * H:] = zr, n
                s["lam"][l] = 1.0 - z
                s["x"][l + 1] = torch.addcmul(x, z, n - x)
        return s
    for l in range(L):
        j = l // 2 if tfm else l
        x = s["x"][l].to(dt)
        y = s["x"][l]
        if rms:
            r = torch.rsqrt((x * x).mean(-1) + EPS)
            s["rinv"][l] = r
            s["y"][l] = x * r.unsqueeze(-1)
            y = s["y"][l]
        if tfm and l % 2 == 0:
            s["qkv"][j] = torch.matmul(y.to(dt), inp["Wqkv"][j].to(dt).t().contiguous())
            q, k, v = _heads_view(case, s["qkv"][j].to(dt), 3)
            P, lse = _probabilities(case, q, k)
            s["attn_o"][j] = _from_heads(case, [torch.matmul(P, v)])
            s["lse"][j] = lse.reshape(-1)
            out = torch.matmul(s["attn_o"][j].to(dt), inp["Wo"][j].to(dt).t().contiguous())
        else:
            a = torch.matmul(y.to(dt), inp["W1"][j].to(dt).t().contiguous())
            s["z"][j], s["dphi"][j] = _gelu(a)
            out = torch.matmul(s["z"][j].to(dt), inp["W2"][j].to(dt).t().contiguous())
        nxt = out + (x if inp["lam"] is None else x * inp["lam"][l].to(dt))
        if post:
            nxt = nxt.to(st).to(dt)
            r = torch.rsqrt((nxt * nxt).mean(-1) + EPS)
            s["rinv"][l] = r
            nxt = nxt * r.unsqueeze(-1)
        s["x"][l + 1] = nxt
    return s


class _Stack64:
    """Gradients of a stack in 64 bits on a given saved state: exact, by k iterations, and of the parameters."""

    def __init__(self, case, inp, state):
        self.c, self.inp, self.s = case, inp, state
        self.f = lambda t: t.to(torch.float64)

    def lam(self, l):
        if self.c["kind"] in CELLS:
            return self.f(self.s["lam"][l])
        return 1.0 if self.inp["lam"] is None else self.f(self.inp["lam"][l])

    def diag(self, l):
        """K_l: the coefficients of the residual path."""
        lam = self.lam(l)
        return lam * self.f(self.s["rinv"][l]).unsqueeze(-1) if self.c["post"] == "rms" else lam

    def through(self, l, G):
        """The gradient with respect to what block l and its residual path add up to, from that of x_{l+1}."""
        if self.c["post"] != "rms":
            return G
        x = self.f(self.s["x"][l + 1])
        return self.f(self.s["rinv"][l]).unsqueeze(-1) * (G - x * (G * x).mean(-1, keepdim=True))

    def inner(self, l, g):
        """Block l's gradient at its inner product: (rows against the second weight, operand of the first, its gradient)."""
        c, s, f = self.c, self.s, self.f
        if c["kind"] == "transformer" and l % 2 == 0:
            j = l // 2
            q, k, v = _heads_view(c, f(s["qkv"][j]), 3)
            P, _ = _probabilities(c, q, k)
            do = _heads_view(c, torch.matmul(g, f(self.inp["Wo"][j])), 1)[0]
            dv = torch.matmul(P.transpose(-1, -2).contiguous(), do)
            dP = torch.matmul(do, v.transpose(-1, -2).contiguous())
            dS = P * (dP - (P * dP).sum(-1, keepdim=True)) / math.sqrt(q.shape[-1])
            return _from_heads(c, [torch.matmul(dS, k), torch.matmul(dS.transpose(-1, -2).contiguous(), q), dv])
        j = l // 2 if c["kind"] == "transformer" else l
        return torch.matmul(g, f(self.inp["W2"][j])) * f(s["dphi"][j])

    def block_vjp(self, l, g):
        c, s, f = self.c, self.s, self.f
        attn = c["kind"] == "transformer" and l % 2 == 0
        j = l // 2 if c["kind"] == "transformer" else l
        dn = torch.matmul(self.inner(l, g), f(self.inp["Wqkv" if attn else "W1"][j]))
        if c["norm"] == "rms":
            y = f(s["y"][l])
            dn = (dn - y * (dn * y).mean(-1, keepdim=True)) * f(s["rinv"][l]).unsqueeze(-1)
        return dn

    # -- recurrent kinds: rows of all steps (or of one) at once ------------------------------------------------
    def rec_inner(self, sl, g):
        """(gradient at the product with W1 [rows, d_ff], direct share of v or None) for the steps of slice sl."""
        c, s, f = self.c, self.s, self.f
        z, x = f(s["z"][sl]), f(s["x"][:-1][sl])
        kind, H = c["kind"], c["d"] // 2 if c["kind"] == "lstm" else c["d"]
        if kind == "rnn":
            return torch.matmul(g, f(self.inp["W2"])) * (1.0 - z * z), None
        if kind == "gated":
            u, cc = z[..., :H], z[..., H:]
            return torch.cat((g * (cc - x) * u * (1 - u), g * u * (1 - cc * cc)), -1), None
        if kind == "lstm":
            i, fg, o, gg = (z[..., q * H:(q + 1) * H] for q in range(4))
            tc = torch.tanh(f(s["x"][1:][sl])[..., :H])
            Gc, Gh, cell = g[..., :H], g[..., H:], x[..., :H]
            thr = Gh * o * (1 - tc * tc)
            dct = Gc + thr
            return torch.cat((dct * gg * i * (1 - i), dct * cell * fg * (1 - fg), Gh * tc * o * (1 - o),
                              dct * i * (1 - gg * gg)), -1), thr * fg
        zz, r, n = (z[..., q * H:(q + 1) * H] for q in range(3))
        dn = g * zz * (1 - n * n)
        drx = torch.matmul(dn, f(self.inp["W1"][2 * H:]))
        return torch.cat((g * (n - x) * zz * (1 - zz), drx * x * r * (1 - r), dn), -1), drx * r

    def rec_vjp(self, sl, g):
        da, direct = self.rec_inner(sl, g)
        kind, H = self.c["kind"], self.c["d"]
        if kind == "gru":
            return torch.matmul(da[..., :2 * H], self.f(self.inp["W1"][:2 * H])) + direct
        v = torch.matmul(da, self.f(self.inp["W1"]))
        return torch.cat((direct, v), -1) if kind == "lstm" else v

    # -- state gradients ------------------------------------------------------------------------------------------
    def e_at(self, l, e):
        if self.c["every"]:
            return self.f(e[l])
        return self.f(e) if l == self.c["L"] else 0.0

    def gradient(self, e, k, exact):
        c = self.c
        L, gamma = c["L"], 0.0 if exact else c["gamma"]
        rec = c["kind"] in RECURRENT
        G = torch.zeros((L + 1, c["N"], c["d"]), dtype=torch.float64, device="cuda")
        G[L] = self.e_at(L, e)
        if exact:
            for l in range(L - 1, -1, -1):
                t = self.through(l, G[l + 1])
                v = self.rec_vjp(slice(l, l + 1), t[None])[0] if rec else self.block_vjp(l, t)
                G[l] = self.lam(l) * t + v + self.e_at(l, e)
            return G
        for l in range(L - 1, -1, -1):
            G[l] = (1 - gamma) * self.diag(l) * G[l + 1] + self.e_at(l, e)
        for _ in range(min(k, L)):
            old = G.clone()
            if rec:
                v = self.rec_vjp(slice(0, L), old[1:])
            for l in range(L - 1, -1, -1):
                if rec:
                    vl = v[l]
                else:
                    t = self.through(l, old[l + 1])
                    vl = self.block_vjp(l, t) + self.lam(l) * t - (1 - gamma) * self.diag(l) * old[l + 1]
                G[l] = (1 - gamma) * self.diag(l) * G[l + 1] + vl + self.e_at(l, e)
        return G

    def kept(self, G):
        """The state gradients as the library keeps them: taken through the norm that made the state."""
        if self.c["post"] == "rms":
            for l in range(1, self.c["L"] + 1):
                G[l] = self.through(l - 1, G[l])
        return G

    def param_grads(self, g):
        c, s, f = self.c, self.s, self.f
        L, N, d = c["L"], c["N"], c["d"]
        tt = lambda a, b: torch.matmul(a.t().contiguous(), b)
        out = {n: torch.zeros(w, dtype=torch.float64, device="cuda") for n, w in _weight_shapes(c).items()}
        if c["kind"] in RECURRENT:
            H = d // 2 if c["kind"] == "lstm" else d
            step = max(1, (1 << 28) // (N * c["d_ff"]))
            for l0 in range(0, L, step):
                sl = slice(l0, min(L, l0 + step))
                da, _ = self.rec_inner(sl, g[1:][sl])
                da, x = da.reshape(-1, c["d_ff"]), f(s["x"][:-1][sl]).reshape(-1, d)
                out["U"] += tt(da, f(self.inp["xin"][sl]).reshape(-1, c["d_in"]))
                if c["kind"] == "gru":
                    z = f(s["z"][sl]).reshape(-1, 3 * H)
                    out["W1"][:2 * H] += tt(da[:, :2 * H], x)
                    out["W1"][2 * H:] += tt(da[:, 2 * H:], z[:, H:2 * H] * x)
                else:
                    out["W1"] += tt(da, x[:, d - H:])
                if c["kind"] == "rnn":
                    out["W2"] += tt(g[1:][sl].reshape(-1, d), f(s["z"][sl]).reshape(-1, c["d_ff"]))
            return out
        for l in range(L):
            attn = c["kind"] == "transformer" and l % 2 == 0
            j = l // 2 if c["kind"] == "transformer" else l
            y = f(s["y"][l] if c["norm"] == "rms" else s["x"][l])
            out["Wqkv" if attn else "W1"][j] = tt(self.inner(l, g[l + 1]), y)
            out["Wo" if attn else "W2"][j] = tt(g[l + 1], f(s["attn_o"][j] if attn else s["z"][j]))
        return out


# ---------------------------------------------------------------------------------------------------------------
# the interface of the measurement
# ---------------------------------------------------------------------------------------------------------------
_STATE = ("x", "y", "rinv", "z", "dphi", "lam", "qkv", "attn_o", "lse")
_OPT = dict(lr=3e-4, beta1=0.9, beta2=0.95, eps=1e-8, weight_decay=0.01, clip_norm=1.0)


def prepare(case, seed):
    inp = _inputs(case, seed)
    dt = _storage(case)
    L, N, d, F, kind = case["L"], case["N"], case["d"], case["d_ff"], case["kind"]
    tfm = kind == "transformer"
    desc = B.make_desc(kind, case["dtype"], case["act"], case["norm"], L, N, d, F, case.get("d_in", 0),
                       lambda_channel=inp["lam"] is not None, lambda_token=kind in CELLS,
                       loss_every_state=case["every"], eps=EPS, gamma=case["gamma"], post=case["post"],
                       heads=case.get("heads", 0), causal=case.get("causal", True), seq_len=case.get("seq_len", 0))
    zeros = lambda shape, t=dt: torch.zeros(shape, dtype=t, device="cuda")
    p = B.Problem(desc=desc, W1=inp["W1"], W2=inp.get("W2"), U=inp.get("U"), lam=inp["lam"], xin=inp.get("xin"),
                  Wqkv=inp.get("Wqkv"), Wo=inp.get("Wo"), e=inp["e"], g=zeros((L + 1, N, d)))
    if case["op"] in ("grad", "exact"):
        for name, t in _forward(case, inp, torch.float32, dt).items():
            setattr(p, name, t)
    else:
        Li = L // 2 if tfm else L
        p.x, p.z = zeros((L + 1, N, d)), zeros((Li, N, F))
        p.x[0] = inp["x0"]
        if case["norm"] == "rms":
            p.y = zeros((L, N, d))
        if case["norm"] == "rms" or case["post"] == "rms":
            p.rinv = zeros((L, N), torch.float32)
        if case["act"] == "gelu":
            p.dphi = zeros((Li, N, F))
        if kind in CELLS:
            p.lam = zeros((L, N, d))
        if tfm:
            p.qkv, p.attn_o = zeros((Li, N, 3 * d)), zeros((Li, N, d))
            p.lse = zeros((Li, N * case["heads"]), torch.float32)
    for name, shape in _weight_shapes(case).items():
        setattr(p, "d" + name, zeros(shape, torch.float32))
    p.workspace = zeros(B.workspace_size(desc), torch.uint8)
    state = {"case": case, "p": p}
    if case["op"] == "train":
        state["target"] = inp["e"]
        p.e = zeros((N, d))
        state["opt"] = B.allocate_optim(p, adamw=True)
        state["step"] = 0
    return state


def _grads(case, p):
    return [p.g] + [getattr(p, "d" + n) for n in _weight_shapes(case)]


def run(state):
    case, p = state["case"], state["p"]
    op = case["op"]
    if op == "train":
        state["step"] += 1
        B.hbp_train_step(p, case["k"], state["target"], B.make_optim("adamw", step=state["step"], **_OPT), state["opt"])
        o = state["opt"]
        return [o.loss, p.x[-1]] + _grads(case, p) + [t for t in o.master if t is not None]
    if op in ("forward", "both"):
        B.hbp_forward(p)
    if op in ("grad", "both"):
        B.hbp_backward(p, case["k"])
    if op == "exact":
        B.hbp_exact_backward(p)
    if op != "forward":
        B.hbp_param_grads(p)
    saved = [getattr(p, n) for n in _STATE if getattr(p, n) is not None and not (n == "lam" and case["kind"] not in CELLS)]
    if op == "forward":
        return saved
    return ([p.x] if op == "both" else []) + _grads(case, p)


def exact(case, seed):
    if work(case)["flops"] > 6e13:
        return None
    inp = _inputs(case, seed)
    op = case["op"]
    f64 = torch.float64
    if op in ("grad", "exact"):
        st = _forward(case, inp, torch.float32, _storage(case))
    else:
        st = _forward(case, inp, f64, f64)
    if op == "forward":
        return [st[n] for n in _STATE if n in st]
    S = _Stack64(case, inp, st)
    e = inp["e"]
    loss = None
    if op == "train":
        diff = st["x"][-1] - e.to(f64)
        loss = (0.5 / case["N"]) * (diff * diff).sum().reshape(1)
        e = diff / case["N"]
    g = S.kept(S.gradient(e, case["k"], op == "exact"))
    dW = S.param_grads(g)
    names = list(_weight_shapes(case))
    out = [g] + [dW[n] for n in names]
    if op == "both":
        return [st["x"]] + out
    if op != "train":
        return out
    o = _OPT
    norm = torch.sqrt(sum((dW[n] ** 2).sum() for n in names))
    clip = torch.clamp(o["clip_norm"] / (norm + 1e-6), max=1.0)
    new = []
    for n in ("W1", "W2", "U", "Wqkv", "Wo"):        # the first update: the bias-corrected moments are g and g^2
        if n in names:
            gr = dW[n] * clip
            new.append(inp[n].to(f64) * (1 - o["lr"] * o["weight_decay"]) - o["lr"] * gr / (gr.abs() + o["eps"]))
    return [loss, st["x"][-1]] + out + new


def _pair_flops(case, l):
    """One product of block l's first weight with its second's shape: flops of the block's contractions, one pass."""
    N, d, F, kind = case["N"], case["d"], case["d_ff"], case["kind"]
    if kind == "transformer" and l % 2 == 0:
        T = case["seq_len"]
        return 2 * N * 4 * d * d, 2 * 2 * N * T * d * (0.5 if case["causal"] else 1.0)
    if kind == "mlp" or kind == "transformer" or kind == "rnn":
        return 2 * N * 2 * d * F, 0
    return 2 * N * F * (d // 2 if kind == "lstm" else d), 0


def work(case):
    L, N, d, F, kind, op = (case[n] for n in ("L", "N", "d", "d_ff", "kind", "op"))
    es = 2 if case["dtype"] == "bf16" else 4
    tfm, rec = kind == "transformer", kind in RECURRENT
    per = [_pair_flops(case, l) for l in range(L)] if not rec else [_pair_flops(case, 0)] * L
    uin = 2 * N * F * case["d_in"] * L if rec else 0
    fwd = sum(a + b for a, b in per) + uin
    its = min(case["k"], L) if op != "exact" else 1
    vjp = sum(sum(a + 2.5 * b for a, b in per[:L - it]) for it in range(its)) if op != "exact" else \
        sum(a + 2.5 * b for a, b in per)
    first = 0.5 if kind in ("mlp", "rnn") else 0.0   # the parameter gradients' own half of a block's VJP
    pg = sum(a * (1 + first) for a, b in per) + uin
    flops = 0.0
    if op in ("forward", "both", "train"):
        flops += fwd
    if op != "forward":
        flops += vjp + pg
    weights = sum(math.prod(s) for s in _weight_shapes(case).values())
    Li = L // 2 if tfm else L
    state = N * d * (L + 1) * es + Li * N * F * es * (2 if case["act"] == "gelu" else 1)
    if case["norm"] == "rms":
        state += L * N * (d * es + 4)
    if kind in CELLS:
        state += L * N * d * es
    if tfm:
        state += Li * N * (4 * d * es + 4 * case["heads"])
    e = N * d * es * (L + 1 if case["every"] else 1)
    nbytes = weights * es + (L * N * case["d_in"] * es if rec else 0) + state
    if op != "forward":
        nbytes += e + (L + 1) * N * d * es + weights * 4
    if op == "train":
        nbytes += weights * (6 * 4 + es)
    return {"bytes": float(nbytes), "flops": float(flops)}


def tolerance(case):
    # about four times the distance from exact() that the cases show
    if case["dtype"] == "f32":
        return {"rel": 3e-6}         # 32-bit sums of up to a thousand terms (seen: 3e-7)
    if case["op"] == "grad":
        return {"rel": 1.2e-2}       # one rounding to bf16 per stored value on a given forward state (seen: 3e-3)
    return {"rel": 2.5e-2}           # the same carried on through the blocks of a forward or exact pass (seen: 4e-3 .. 9e-3)
