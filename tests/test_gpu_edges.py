"""GPU parity at the sizes where a kernel's tiling can go wrong: one element past a tile, one short of it, the smallest
call, and the sizes at which a dispatch changes kernels.  Same oracle and bars as test_gpu_parity."""
import numpy as np
import pytest

from oracle import hbp_oracle as O
from paper_2501_17086_amd import synth
from tests import helpers as H
from tests.test_gpu_parity import B, W, _check_backward, _setup  # noqa: F401  (B is the fixture)

pytestmark = pytest.mark.gpu


def _forward_matches(B, w):
    inp, st, sv, p = _setup(B, w)
    B.hbp_forward(p)
    for l in range(w.L + 1):
        H.assert_close(H.to_np(p.x)[l], sv["x"][l], H.TOL[w.dtype], f"{w.name} x[{l}]")
    return inp, st, sv, p


# tokens, width, inner width: around the 64- and 128-wide output tiles and the 64- and 32-deep slices (a contraction that
# ends inside a slice), enough tiles for the 128-wide ones (2 blocks x 23 x 8 of them), and two rounds of whole 256-wide
# tiles plus remainders of rows and columns in launches of their own
@pytest.mark.parametrize("N,d,d_ff", [(1, 8, 8), (7, 56, 64), (63, 64, 72), (65, 72, 128), (127, 120, 136),
                                      (129, 128, 264), (191, 136, 1032), (2900, 264, 1000), (8200, 512, 2056)])
def test_products_around_the_tile_edges(B, N, d, d_ff):
    w = synth.scaled(W["resnet_like"], name=f"mlp_{N}_{d}_{d_ff}", L=2, N=N, d=d, d_ff=d_ff, w2_scale=0.7, ks=(1,))
    inp, st, sv, p = _forward_matches(B, w)
    H.assert_close(H.to_np(p.z), sv["z"], H.TOL["bf16"], f"{w.name} z")
    H.assert_close(H.to_np(p.dphi), sv["dphi"], H.TOL["bf16"], f"{w.name} act'")
    _check_backward(B, w, p, st, sv, inp, w.name)


# few tiles, the wavefronts sharing the contraction: 64 x 32 tiles (257 to 512 blocks of 32 x 32) and 32 x 32 ones, contractions
# of one to 17 slices of 64 (wavefronts with none, with one more than others, with a last slice that ends inside), tokens,
# widths and inner widths that end inside a tile
@pytest.mark.parametrize("N,d,d_ff", [(1000, 328, 1304), (520, 1032, 72), (250, 520, 1096), (33, 1096, 264), (640, 512, 200),
                                      (96, 40, 1288)])
def test_products_of_few_tiles(B, N, d, d_ff):
    w = synth.scaled(W["resnet_like"], name=f"mlp_{N}_{d}_{d_ff}", L=2, N=N, d=d, d_ff=d_ff, w2_scale=0.7, ks=(1,))
    inp, st, sv, p = _forward_matches(B, w)
    H.assert_close(H.to_np(p.z), sv["z"], H.TOL["bf16"], f"{w.name} z")
    _check_backward(B, w, p, st, sv, inp, w.name)


# several products in one launch (a transformer's first and second contractions in pairs, its four parameter gradients), on each kind
# of tile: 32 x 32, 64 x 32, 64 x 64 and 128 x 128, products of one tile beside larger ones, sizes that end inside a tile and a slice; the
# second contractions in tiles of 128: 240, of 4096 and more 220 (a tile per compute unit) and, apart, 264; of 2056 660 (together) and 880
@pytest.mark.parametrize("dtype,N,T,d,d_ff", [("bf16", 9, 9, 16, 8), ("bf16", 40, 8, 64, 72), ("bf16", 200, 40, 136, 264),
                                              ("bf16", 520, 40, 200, 1032), ("bf16", 1000, 40, 264, 1096), ("bf16", 2960, 40, 520, 2056),
                                              ("bf16", 1520, 40, 520, 2056), ("bf16", 520, 40, 1368, 4104), ("bf16", 680, 40, 1368, 4104),
                                              ("bf16", 4200, 40, 520, 2056), ("bf16", 5600, 40, 520, 2056),
                                              ("f32", 9, 9, 16, 8), ("f32", 120, 40, 72, 264)])
def test_products_in_one_launch(B, dtype, N, T, d, d_ff):
    w = synth.scaled(W["gpt2_paper"], name=f"tfm_{dtype}_{N}_{d}_{d_ff}", L=4, N=N, seq_len=T, d=d, heads=1 if d < 64 else d // 8,
                     d_ff=d_ff, dtype=dtype, w1_std=0.0, w2_std=0.0, w2_scale=0.6, ks=(1, 2))
    inp, st, sv, p = _forward_matches(B, w)
    _check_backward(B, w, p, st, sv, inp, w.name, exact=False)


# 128 x 128 tiles with contractions that end inside a slice: 192 to 256 of them (slices of 64: the block VJPs of the first, the
# forward of the second, the parameter gradients of the last), 400 and 450 (four stages), 512 and more (three workgroups per
# compute unit: the VJPs of the third, the forward of the fourth)
@pytest.mark.parametrize("N,d,d_ff", [(1500, 1000, 1096), (3100, 1000, 1096), (4200, 1000, 1096), (8200, 1000, 1096),
                                      (104, 1288, 1288)])
def test_products_on_wide_tiles(B, N, d, d_ff):
    w = synth.scaled(W["resnet_like"], name=f"mlp_{N}_{d}_{d_ff}", L=2, N=N, d=d, d_ff=d_ff, w2_scale=0.7, ks=(1,))
    inp, st, sv, p = _forward_matches(B, w)
    H.assert_close(H.to_np(p.z), sv["z"], H.TOL["bf16"], f"{w.name} z")
    _check_backward(B, w, p, st, sv, inp, w.name)


# head widths around the 32, 64 and 128 columns that the matrix-core kernels pad to (136: the plain kernels), on sequence
# lengths of one ragged tile, one workgroup, past the whole-problem kernels (128 / 256 positions) and past a block of tiles
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("dh,T", [(8, 33), (16, 1), (24, 128), (32, 100), (32, 300), (40, 129), (56, 257), (64, 192), (72, 65),
                                  (104, 161), (128, 32), (128, 128), (128, 200), (136, 40)])
def test_attention_head_widths(B, dh, T, causal):
    w = synth.scaled(W["gpt2_paper"], name=f"tfm_dh{dh}_T{T}", L=2, N=3 * T, seq_len=T, d=2 * dh, heads=2, d_ff=64, w1_std=0.0,
                     w2_std=0.0, w2_scale=0.6, causal=causal, ks=(1, 2))
    inp, st, sv, p = _forward_matches(B, w)
    H.assert_close(H.to_np(p.attn_o), sv["o"][0::2], H.TOL["bf16"], f"{w.name} attention output")
    _check_backward(B, w, p, st, sv, inp, w.name, exact=False)


# problems enough that a workgroup's wavefronts take a tile each (above), fewer, so that they share one's tiles, and the numbers at
# which that changes (256 or 512 tiles), on widths with one, two and four blocks of columns
@pytest.mark.parametrize("dh,heads,seqs,T,causal", [(24, 4, 26, 257, True), (40, 4, 26, 257, False), (64, 4, 16, 300, True),
                                                    (104, 3, 20, 290, False), (128, 2, 30, 290, True), (32, 2, 32, 256, True),
                                                    (32, 2, 33, 256, True), (64, 2, 16, 250, False), (64, 2, 17, 250, False),
                                                    (64, 1, 1, 1000, True), (128, 1, 1, 520, False), (48, 1, 2, 513, True)])
def test_attention_with_shared_tiles(B, dh, heads, seqs, T, causal):
    w = synth.scaled(W["gpt2_paper"], name=f"tfm_dh{dh}_T{T}_x{heads * seqs}", L=2, N=seqs * T, seq_len=T, d=heads * dh, heads=heads,
                     d_ff=64, w1_std=0.0, w2_std=0.0, w2_scale=0.6, causal=causal, ks=(1,))
    inp, st, sv, p = _forward_matches(B, w)
    H.assert_close(H.to_np(p.attn_o), sv["o"][0::2], H.TOL["bf16"], f"{w.name} attention output")
    _check_backward(B, w, p, st, sv, inp, w.name, exact=False)


_KINDS = {"rnn": ("gated_rnn_contractive", 1, 1), "token": ("gated_rnn_token_gates", 1, 1), "gated": ("gru_cell", 1, 2),
          "lstm": ("lstm_cell", 2, 4), "gru": ("gru_std_cell", 1, 3)}


def _chain(kind, L, N, H, inner=None, **kw):
    base, dm, fm = _KINDS[kind]
    return synth.scaled(W[base], name=f"{kind}_{L}_{N}_{H}", L=L, N=N, d=dm * H, d_ff=fm * (inner or H), d_in=16, ks=(1,), **kw)


# chains along time in one launch: widths around a workgroup's 32 channels, the quarters of a contraction and the register
# sizes (256 / 512 / 1024), batches around 16-row groups, chains of one step and of more than the four slots; 64 rows at
# width 1024 take two row tiles per workgroup; 65 rows at that width and widths past 1024 go step by step
@pytest.mark.parametrize("kind,L,N,H", [("rnn", 1, 1, 8), ("rnn", 9, 17, 264), ("rnn", 6, 64, 1024), ("token", 7, 15, 72),
                                        ("gated", 2, 16, 32), ("gated", 9, 33, 136), ("gated", 5, 65, 1024), ("lstm", 1, 5, 24),
                                        ("lstm", 9, 16, 520), ("lstm", 6, 64, 1024), ("gru", 3, 1, 40), ("gru", 9, 31, 256),
                                        ("gru", 6, 48, 1000), ("gru", 4, 8, 1032),
                                        # from 12 steps on: groups on one XCD, of 8 rows or of 16
                                        ("rnn", 13, 17, 264), ("rnn", 12, 144, 224), ("token", 12, 9, 40), ("gated", 14, 33, 136),
                                        ("lstm", 12, 20, 520), ("gru", 13, 31, 256), ("gru", 12, 40, 1000)])
def test_chains_along_time(B, kind, L, N, H):
    w = _chain(kind, L, N, H)
    inp, st, sv, p = _forward_matches(B, w)
    _check_backward(B, w, p, st, sv, inp, w.name)


# the fifth wavefront's reading ahead: chains shorter and longer than the four steps it is ahead by, widths whose last block of 32 channels
# and last piece of 16 inputs end inside, the rows past the batch, with and without it (the gated cell's two rows; width 1024; the
# GRU's 80 workgroups)
@pytest.mark.parametrize("kind,L,N,H", [("rnn", 12, 3, 8), ("rnn", 13, 33, 504), ("token", 17, 3, 264), ("gated", 16, 2, 24),
                                        ("gated", 16, 3, 24), ("gated", 12, 17, 1000), ("lstm", 15, 9, 488), ("gru", 12, 65, 56),
                                        ("gru", 14, 7, 504), ("gru", 12, 32, 504), ("gru", 12, 33, 504)])
def test_chains_that_read_ahead(B, kind, L, N, H):
    w = _chain(kind, L, N, H)
    inp, st, sv, p = _forward_matches(B, w)
    _check_backward(B, w, p, st, sv, inp, w.name)


@pytest.mark.parametrize("d,d_ff,act", [(40, 296, "tanh"), (296, 40, "tanh"), (64, 64, "identity")])
def test_chains_along_time_of_two_widths(B, d, d_ff, act):
    w = synth.scaled(W["gated_rnn_contractive"], name=f"rnn_{d}_{d_ff}_{act}", L=7, N=20, d=d, d_ff=d_ff, d_in=16, act=act,
                     loss_every_state=act == "tanh", ks=(1,))
    inp, st, sv, p = _forward_matches(B, w)
    _check_backward(B, w, p, st, sv, inp, w.name)


@pytest.mark.parametrize("kind", ["rnn", "gated", "lstm", "gru"])
def test_chains_along_time_with_nan_rows_and_on_two_streams(B, kind):
    """A row of NaNs of the pattern that marks an empty exchange slot runs through the chain as NaN and leaves the other
    rows what they are without it; two chains at once on streams of their own do not disturb each other."""
    import torch
    w = _chain(kind, 12, 20, 64)
    inp, st, sv, p = _setup(B, w)
    q = B.allocate(w, inp)
    q.x[0].view(torch.int16)[3] = -1
    torch.cuda.synchronize()
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    for b, s in ((p, s1), (q, s2)):
        B.hbp_forward(b, stream=s.cuda_stream)
        B.hbp_exact_backward(b, stream=s.cuda_stream)
    torch.cuda.synchronize()
    keep = [n for n in range(w.N) if n != 3]
    assert torch.equal(p.x[:, keep], q.x[:, keep]) and torch.equal(p.g[:, keep], q.g[:, keep])
    assert bool(q.x[1:, 3].isnan().all()) and not bool(p.x.isnan().any())


@pytest.mark.parametrize("L", [9, 13])           # groups anywhere, groups on one XCD
@pytest.mark.parametrize("kind,H", [("rnn", 264), ("gated", 64), ("lstm", 72), ("gru", 256)])
def test_chains_along_time_in_a_graph(B, kind, H, L):
    """Forward and exact backpropagation recorded into a HIP graph: every replay, with eager chains and synchronisations
    between them, gives the eager result bit for bit."""
    import torch
    w = _chain(kind, L, 20, H)
    inp, st, sv, p = _setup(B, w)

    def both():
        B.hbp_forward(p)
        B.hbp_exact_backward(p)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        both()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    want = [t.clone() for t in (p.x, p.z, p.g)]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        both()
    for _ in range(3):
        p.x[0] += 1
        both()                                   # eager chains of other values between the replays
        torch.cuda.synchronize()
        p.x[0].copy_(want[0][0])
        p.g.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip((p.x, p.z, p.g), want))


# An infinity in the last block of 32 channels, at widths whose quarters of the contraction reach past it: saturated gates
# stay finite, and gradients are infinite, not NaN.  It meets one step's product, so that what follows does not mix the two.
# (wait: groups anywhere, as such a short chain has them, and on one XCD, where two blocks share an operand)
@pytest.mark.parametrize("wait", [0, 4])
@pytest.mark.parametrize("kind", ["rnn", "token", "gated", "lstm", "gru"])
@pytest.mark.parametrize("H_", [24, 72, 264, 600])
def test_chains_along_time_with_infinities(B, kind, H_, wait):
    import torch
    w = _chain(kind, 2, 5, H_)
    inp, st, _, p = _setup(B, w)
    c = w.d - 3                                    # (the LSTM's hidden part comes second)
    inp["x0"][2, c] = np.inf
    p.x[0, 2, c] = float("inf")
    # positive weights of that channel: what it meets saturates upwards, the standard GRU's reset gate among it
    col = H_ - 3
    inp["W1"][:, col] = np.abs(inp["W1"][:, col]) + 2.0 ** -7
    p.W1.copy_(torch.from_numpy(inp["W1"]))
    st = H.oracle_stack(w, inp)
    with np.errstate(invalid="ignore", over="ignore"):
        sv = O.forward(st, inp["x0"], inp["xin"])
        _run_chain(B, p, 1, wait)
        _same_numbers(H.to_np(p.x)[1], sv["x"][1], f"{w.name} x[1]")
        # backward on a finite state
        inp["x0"][2, c], p.x[0, 2, c] = 0, 0
        sv = O.forward(st, inp["x0"], inp["xin"])
        _run_chain(B, p, 1, wait)
        inp["e"][1, 2, c] = np.inf
        p.e[1, 2, c] = float("inf")
        _run_chain(B, p, 0, wait)
        _same_numbers(H.to_np(p.g)[0], O.exact_backward(st, sv, inp["e"])[0], f"{w.name} g[0]")


def _same_numbers(got, want, what):
    assert np.array_equal(np.isnan(got), np.isnan(want)), f"{what}: NaN"
    inf = np.isinf(want)
    assert np.array_equal(np.isinf(got), inf) and np.array_equal(got[inf], want[inf]), f"{what}: infinities"
    H.assert_close(np.where(np.isfinite(want), got, 0), np.where(np.isfinite(want), want, 0), H.TOL["bf16"], what)


# Groups whose workgroups do not get to run side by side are left to one workgroup: all of them (wait 2), or those whose
# workgroups do not all start at the same moment (wait 1).  The same results bit for bit.
@pytest.mark.parametrize("wait", [1, 2])
@pytest.mark.parametrize("kind,L,N,H", [("rnn", 1, 1, 8), ("rnn", 9, 17, 264), ("rnn", 6, 64, 1024), ("token", 7, 15, 72),
                                        ("gated", 9, 33, 136), ("gated", 6, 64, 1000), ("lstm", 1, 5, 24), ("lstm", 9, 16, 520),
                                        ("lstm", 6, 64, 1024), ("gru", 3, 1, 40), ("gru", 9, 31, 256), ("gru", 6, 64, 1024)])
def test_chains_along_time_by_one_workgroup(B, kind, L, N, H, wait):
    import ctypes as C
    import torch
    w = _chain(kind, L, N, H)
    inp, st, sv, p = _setup(B, w)
    q = B.allocate(w, inp)
    B.hbp_forward(p)
    b = q.buffers()
    f = B.lib().hbp_internal_chains
    s = torch.cuda.current_stream().cuda_stream
    assert f(C.byref(q.desc), 1, wait, C.byref(b), C.c_void_p(s)) == B.HBP_OK
    for n in ("x", "z", "lam"):
        assert torch.equal(getattr(p, n), getattr(q, n)), n
    B.hbp_exact_backward(p)
    assert f(C.byref(q.desc), 0, wait, C.byref(b), C.c_void_p(s)) == B.HBP_OK
    assert torch.equal(p.g, q.g)


ANYWHERE, ON_XCD = 3, 4


def _run_chain(B, p, forward, wait):
    import ctypes as C
    import torch
    b = p.buffers()
    f = B.lib().hbp_internal_chains
    assert f(C.byref(p.desc), forward, wait, C.byref(b), C.c_void_p(torch.cuda.current_stream().cuda_stream)) == B.HBP_OK


def _groups_on_xcd(B, p):
    """Per group on one XCD of p's last chain how many workgroups have started and whether it was given up; workgroups of each."""
    import ctypes as C
    import torch
    n, m, o = C.c_int(), C.c_int(), C.c_size_t()
    assert B.lib().hbp_internal_chain_groups(C.byref(p.desc), C.byref(n), C.byref(m), C.byref(o)) == B.HBP_OK
    torch.cuda.synchronize()
    words = p.workspace[o.value:o.value + 4 * n.value].view(torch.int32).cpu().numpy().astype(np.uint32)
    return words & 0x7FFFFFFF, words >> 31 == 1, m.value


# Groups on one XCD each (of 8 rows, or of 16 where there would be too many) against groups whose workgroups may be anywhere
# (of 16 or 32 rows): the same results bit for bit, and the former did all of it.  Odd numbers of blocks, a last group with one row,
# more groups than XCDs, the widest with every compute unit taken; chains of one step and of more than the four slots.
@pytest.mark.parametrize("kind,L,N,H", [("rnn", 13, 1, 8), ("rnn", 2, 9, 96), ("rnn", 12, 1030, 32), ("token", 12, 96, 672), ("token", 15, 33, 520),
                                        ("rnn", 6, 144, 224), ("gated", 12, 65, 512), ("gated", 13, 17, 40), ("lstm", 12, 64, 1024),
                                        ("lstm", 14, 25, 264), ("lstm", 5, 144, 224), ("gru", 12, 96, 672), ("gru", 15, 31, 1000),
                                        ("gru", 12, 64, 1024), ("gru", 2, 126, 512)])
def test_chains_on_one_xcd_and_anywhere(B, kind, L, N, H):
    import torch
    w = _chain(kind, L, N, H)
    inp, st, sv, p = _setup(B, w)
    q = B.allocate(w, inp)
    for forward in (1, 0):
        p.workspace.zero_()
        _run_chain(B, p, forward, ON_XCD)
        started, gone, members = _groups_on_xcd(B, p)
        assert (started == members).all() and not gone.any()
        _run_chain(B, q, forward, ANYWHERE)
    for n in ("x", "z", "lam", "g"):
        assert torch.equal(getattr(p, n), getattr(q, n)), n


# Some groups on one XCD are given up before they start, as where other kernels hold its compute units: the second launch does them
# again, together with those that share a larger group of its own, and leaves out the larger groups of which all is done.  Groups
# of 8 rows in larger ones of 16 and 32, of 16 in 16 and 32; none, some and all given up; a last larger group that is not whole.
@pytest.mark.parametrize("gone", [0x0002, 0x4921, 0x00F0, 0xFFFF])
@pytest.mark.parametrize("kind,L,N,H", [("rnn", 9, 76, 96), ("token", 6, 64, 1024), ("rnn", 5, 144, 224), ("token", 3, 96, 672),
                                        ("gated", 6, 76, 96), ("gated", 5, 58, 1000), ("lstm", 6, 64, 1024), ("lstm", 7, 70, 264),
                                        ("lstm", 3, 96, 672), ("gru", 7, 76, 96), ("gru", 6, 64, 1024), ("gru", 5, 90, 672),
                                        ("gru", 1, 144, 224)])
def test_chains_of_which_groups_on_one_xcd_are_given_up(B, kind, L, N, H, gone):
    import torch
    w = _chain(kind, L, N, H)
    inp, st, sv, p = _setup(B, w)
    q = B.allocate(w, inp)
    for forward in (1, 0):
        p.workspace.zero_()
        _run_chain(B, p, forward, ON_XCD | gone << 8)
        started, given_up, members = _groups_on_xcd(B, p)
        want = np.array([bool(gone >> (j % 16) & 1) for j in range(len(started))])
        assert np.array_equal(given_up, want) and (started[~want] == members).all()
        _run_chain(B, q, forward, ANYWHERE)
    for n in ("x", "z", "lam", "g"):
        assert torch.equal(getattr(p, n), getattr(q, n)), n


# Four chains at once, each as wide as the chip: some groups do not get together on an XCD and are left to the second launch.
@pytest.mark.parametrize("kind,N,H", [("rnn", 64, 1024), ("lstm", 128, 512), ("gru", 64, 1024)])
def test_four_chains_at_once(B, kind, N, H):
    import torch
    w = _chain(kind, 40, N, H)
    inp, st, sv, p = _setup(B, w)
    B.hbp_forward(p)
    B.hbp_exact_backward(p)
    others = [(B.allocate(w, inp), torch.cuda.Stream()) for _ in range(4)]
    torch.cuda.synchronize()
    for step in (B.hbp_forward, B.hbp_exact_backward):
        for q, s in others:
            step(q, stream=s.cuda_stream)
    torch.cuda.synchronize()
    for q, _ in others:
        for n in ("x", "z", "lam", "g"):
            assert n == "lam" and p.lam is None or torch.equal(getattr(p, n), getattr(q, n)), n


# fp32 products: around the 32- and 64-wide tiles, contractions that end inside a chunk of 32 or leave a wavefront's
# quarter empty, and enough blocks (40 x 4 x 4 tiles of 64) for the wide tiles
@pytest.mark.parametrize("L,N,d,d_ff", [(2, 1, 8, 8), (2, 31, 40, 24), (3, 65, 32, 72), (2, 130, 264, 136), (40, 250, 72, 232)])
def test_fp32_products_around_the_tile_edges(B, L, N, d, d_ff):
    w = synth.scaled(W["mlp_small_f32"], name=f"f32_{N}_{d}_{d_ff}", L=L, N=N, d=d, d_ff=d_ff, norm="rms", lam="uniform",
                     lam_lo=0.9, lam_hi=1.0, w2_scale=1 / np.sqrt(L), ks=(1, 2))
    inp, st, sv, p = _forward_matches(B, w)
    H.assert_close(H.to_np(p.dphi), sv["dphi"], H.TOL["f32"], f"{w.name} act'")
    _check_backward(B, w, p, st, sv, inp, w.name)


# whole 256-wide tiles (144 of them), contractions of three (too few for the early loads of the fused operand), four and
# five slices of 32, in pairs of slices (an even number) and singly
@pytest.mark.parametrize("d", [96, 128, 160])
def test_short_contractions_on_whole_tiles(B, d):
    w = synth.scaled(W["resnet_like"], name=f"mlp_short_{d}", L=2, N=4608, d=d, d_ff=1024, w2_scale=0.7, ks=(1,))
    inp, st, sv, p = _forward_matches(B, w)
    H.assert_close(H.to_np(p.z), sv["z"], H.TOL["bf16"], f"{w.name} z")
    H.assert_close(H.to_np(p.dphi), sv["dphi"], H.TOL["bf16"], f"{w.name} act'")
    _check_backward(B, w, p, st, sv, inp, w.name)


# Two and more whole 256-wide tiles per workgroup, with contractions of five and seven slices (an odd number: singly), so that the
# waits after an epilogue count its operations: the fused operands of the backward pass (narrow d), of the residual sum
# (narrow d_ff) and GELU.  Then products of 512 whole tiles in one matrix with remainders of rows and columns, whose parts
# start inside the second output and the coefficients per channel.
@pytest.mark.parametrize("N,d,d_ff,act", [(33280, 160, 1024, "gelu"), (33280, 224, 1024, "tanh"), (33280, 1024, 160, "gelu"),
                                          (16640, 2048, 224, "gelu"), (16400, 512, 2056, "gelu"), (16400, 2056, 128, "gelu")])
def test_several_tiles_per_workgroup(B, N, d, d_ff, act):
    w = synth.scaled(W["resnet_like"], name=f"mlp_{N}_{d}_{d_ff}", L=1, N=N, d=d, d_ff=d_ff, w2_scale=0.7, act=act, ks=(1,))
    inp, st, sv, p = _forward_matches(B, w)
    H.assert_close(H.to_np(p.z), sv["z"], H.TOL["bf16"], f"{w.name} z")
    if act == "gelu":
        H.assert_close(H.to_np(p.dphi), sv["dphi"], H.TOL["bf16"], f"{w.name} act'")
    B.hbp_exact_backward(p)
    H.assert_close(H.to_np(p.g)[0], O.exact_backward(st, sv, inp["e"])[0], H.TOL["bf16"], f"{w.name} g[0]")


# parameter gradients whose contraction is shared out unequally (193 slices of 32 in 3 shares, 258 in 4, 321 in 5), on the
# kernels of small tiles, and the sum of 3, 4 and 5 shares
@pytest.mark.parametrize("L,N,d,d_ff", [(2, 6176, 256, 256), (2, 8256, 256, 512), (1, 10272, 512, 256)])
def test_unequal_shares_of_a_contraction(B, L, N, d, d_ff):
    w = synth.scaled(W["resnet_like"], name=f"mlp_{N}_{d}_{d_ff}", L=L, N=N, d=d, d_ff=d_ff, w2_scale=0.7, ks=(1,))
    inp, st, sv, p = _forward_matches(B, w)
    _check_backward(B, w, p, st, sv, inp, w.name)


# The same on the 256 x 256 kernel: 257 and 258 slices in 4 shares, 257 in 4 over 4 blocks and in 2 over 2 blocks that are taken one
# at a time, 513 in 4 over 3 blocks (768 tiles, three for a workgroup).  Against 64-bit products of what the call read; dW2 is sums
# of exact products, in 32 bits over 16416 tokens: 1e-5 (the root of their number times 2^-24 is 8e-6).
@pytest.mark.parametrize("L,N,d,d_ff,shares", [(1, 8224, 1024, 4096, 4), (1, 8256, 1024, 4096, 4), (4, 8224, 512, 2048, 4),
                                               (2, 8224, 1024, 4096, 2), (3, 16416, 1024, 4096, 4)])
def test_unequal_shares_on_whole_tiles(B, L, N, d, d_ff, shares):
    import torch
    w = synth.scaled(W["resnet_like"], name=f"mlp_{L}_{N}_{d}_{d_ff}", L=L, N=N, d=d, d_ff=d_ff, w2_scale=0.7, ks=(1,))
    inp = synth.make_inputs(w)
    p = B.allocate(w, inp)
    fewer = B.hbp_desc.from_buffer_copy(p.desc)
    fewer.N = 2048                                   # (no shares: what is left of the workspace are the partial sums)
    assert round((B.workspace_size(p.desc) - B.workspace_size(fewer) * N / 2048) / (L * d * d_ff * 4)) == shares
    B.hbp_forward(p)
    B.hbp_backward(p, 1)
    B.hbp_param_grads(p)
    for l in range(L):
        g, W2 = p.g[l + 1].double(), p.W2[l].double()
        H.assert_close(H.to_np(p.dW2)[l], (g.T @ p.z[l].double()).cpu().numpy(), 1e-5, f"{w.name} dW2[{l}]")
        da = ((g @ W2) * p.dphi[l].double()).to(torch.bfloat16).double()
        H.assert_close(H.to_np(p.dW1)[l], (da.T @ p.y[l].double()).cpu().numpy(), H.TOL["bf16"], f"{w.name} dW1[{l}]")


# the scan of rows with a norm: widths around the chunks of 512 (a last chunk of one vector, of all but one, none), one to nine
# layers (fewer than the three that are loaded ahead, and every remainder), fewer rows than a workgroup's four, more rows
# than the line for whole chunks, coefficients of 1 and per channel
@pytest.mark.parametrize("lam", ["one", "uniform"])
@pytest.mark.parametrize("L,N,d", [(1, 3, 40), (3, 5, 520), (4, 1, 8), (5, 7, 504), (6, 33, 512), (7, 9, 520), (9, 6, 1016),
                                   (5, 2, 1024), (6, 5, 1032), (4, 3, 1544), (8, 5, 2040), (4, 4100, 512), (4, 2, 2056)])
def test_scan_of_rows(B, L, N, d, lam):
    w = synth.scaled(W["resnet_like"], name=f"rows_{L}_{N}_{d}_{lam}", L=L, N=N, d=d, d_ff=16, lam=lam, w2_scale=0.7, ks=(1, 2))
    inp, st, sv, p = _forward_matches(B, w)
    _check_backward(B, w, p, st, sv, inp, w.name)


# the same in fp32, and on both sides of the lines up to which few rows of a ragged width take the pipelined form (a layer of 4 MB,
# 6144 rows in bf16 and 4096 in fp32; more rows of narrow widths in bf16, over eight layers with coefficients per channel)
@pytest.mark.parametrize("dtype,L,N,d", [("f32", 4, 3, 40), ("f32", 5, 9, 504), ("f32", 7, 6, 512), ("f32", 6, 5, 520), ("f32", 5, 3, 1024),
                                         ("f32", 4, 4096, 40), ("f32", 4, 4100, 40), ("f32", 5, 2048, 512), ("f32", 4, 2049, 520),
                                         ("f32", 4, 5, 1544), ("bf16", 4, 6144, 136), ("bf16", 7, 6200, 136), ("bf16", 8, 6200, 136),
                                         ("bf16", 4, 4200, 504), ("bf16", 4, 2100, 1000)])
def test_scan_of_rows_around_the_lines_of_its_forms(B, dtype, L, N, d):
    w = synth.scaled(W["resnet_like"], name=f"rows_{dtype}_{L}_{N}_{d}", dtype=dtype, L=L, N=N, d=d, d_ff=16, w2_scale=0.7, ks=(1,))
    inp, st, sv, p = _forward_matches(B, w)
    _check_backward(B, w, p, st, sv, inp, w.name)


# the norm's kernels: rows held by 16, 32 or 64 lanes and one to eight vectors per lane, the last partly past the width, and
# a row count that leaves part of a wavefront without rows; in front of the block (y, rinv) and after the sum, in place
@pytest.mark.parametrize("post", ["none", "rms"])
@pytest.mark.parametrize("d,N", [(8, 1), (128, 33), (136, 5), (256, 17), (264, 7), (512, 3), (520, 9), (1024, 2), (1032, 6),
                                 (2056, 5), (4096, 3)])
def test_row_norms(B, d, N, post):
    w = synth.scaled(W["resnet_like"], name=f"norm_{d}_{N}_{post}", L=2, N=N, d=d, d_ff=16, w2_scale=0.7, post=post,
                     norm="rms" if post == "none" else "none", ks=(0,))
    inp, st, sv, p = _forward_matches(B, w)
    H.assert_close(H.to_np(p.rinv), sv["rpost" if post == "rms" else "rinv"], H.TOL["bf16"], f"{w.name} rinv")
    if post == "none":
        H.assert_close(H.to_np(p.y), sv["y"], H.TOL["bf16"], f"{w.name} y")


# the scan of w^0 where its states are shared out inside a workgroup: chains around a segment, a block of segments and two of them
# (8 of one state, 8 of two, 32 of two, 64 of four), 64-channel slabs that end inside, and the first sizes that keep other forms
@pytest.mark.parametrize("L,N,d", [(1, 3, 40), (2, 1, 8), (8, 9, 40), (9, 5, 56), (16, 3, 8), (17, 7, 72), (31, 129, 520), (7, 300, 720), (7, 320, 720), (33, 9, 40),
                                   (64, 3, 104), (65, 20, 200), (130, 64, 512), (257, 33, 2048), (256, 3, 72), (257, 5, 8),
                                   (513, 2, 136), (1100, 1, 64), (40, 513, 1024), (20, 1030, 1024), (40, 24, 2048),
                                   (35, 32, 2048)])
@pytest.mark.parametrize("dtype,lam,every,gamma", [("bf16", "token", True, 0.0), ("bf16", "channel", True, 0.3),
                                                   ("bf16", "one", False, 0.02), ("f32", "channel", False, 0.0),
                                                   ("f32", "token", True, 0.0), ("f32", "one", True, 0.1)])
def test_scan_with_its_states_shared_out(B, L, N, d, dtype, lam, every, gamma):
    import torch
    if L * N * d > (1 << 24) and (dtype == "f32" or lam == "one"):
        pytest.skip("the large sizes in bf16 with coefficients only: the oracle takes the time")
    st = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator().manual_seed(L + N + d)
    lo = 0.6 if every else 0.97                    # (without a source a thousand coefficients leave something)
    rand = lambda *s: torch.rand(s, generator=gen) * (1 - lo) + lo
    e = torch.randn((L + 1, N, d) if every else (N, d), generator=gen).to(st)
    lm = {"token": lambda: rand(L, N, d).to(st), "channel": lambda: rand(L, d), "one": lambda: None}[lam]()
    desc = B.make_desc("rnn", dtype, "tanh", "none", L, N, d, 8, 8, lambda_channel=lam == "channel", lambda_token=lam == "token",
                       loss_every_state=every, gamma=gamma)
    z = lambda *s: torch.zeros(s, dtype=st, device="cuda")
    p = B.Problem(desc=desc, W1=z(8, d), W2=z(d, 8), U=z(8, 8), lam=None if lm is None else lm.cuda(), xin=None, e=e.cuda(),
                  g=torch.full((L + 1, N, d), float("nan"), dtype=st, device="cuda"))
    p.workspace = torch.zeros(B.workspace_size(desc), dtype=torch.uint8, device="cuda")
    B.hbp_initial_estimate(p, "auto")
    torch.cuda.synchronize()
    a = np.zeros((L + 1, N, d))
    a[:] = e.double().numpy() if every else 0
    a[L] = e[L].double().numpy() if every else e.double().numpy()
    rows = [(1 - gamma) * (np.ones((1, d)) if lm is None else lm[l].double().numpy()) for l in range(L)]
    want = O.cumsumprod_reverse(a, lambda l: rows[l])
    for l in range(L + 1):
        H.assert_close(H.to_np(p.g)[l], want[l], H.TOL[dtype], f"state {l}")


def _walk(a, lam, top):
    """Every state of g_l = lam_l g_{l+1} + a_l in float32, one after the other."""
    g = [np.asarray(top, np.float32)]
    for l in range(len(lam) - 1, -1, -1):
        g.append((lam[l].astype(np.float64) * g[-1] + a[l]).astype(np.float32))
    return np.stack(g[::-1])


# the same scan with infinities, NaNs, coefficients of zero, above one and so large or small that the product of a segment's leaves the
# range of fp32: what comes out is what the walk from state to state gives, in every segment below too.  Chains of each form (segments of
# one, two and four states), a column of its own for each case, others of ordinary numbers beside it.
@pytest.mark.parametrize("L", [7, 21, 100, 300])
@pytest.mark.parametrize("dtype,lam", [("bf16", "token"), ("bf16", "channel"), ("f32", "token"), ("f32", "channel")])
def test_scan_of_segments_with_special_values(B, L, dtype, lam):
    import torch
    st = torch.bfloat16 if dtype == "bf16" else torch.float32
    N, d = 3, 136
    gen = torch.Generator().manual_seed(L)
    e = torch.randn((L + 1, N, d), generator=gen)
    lm = torch.rand((L, N, d) if lam == "token" else (L, d), generator=gen) * 0.4 + 0.6
    inf, m = float("inf"), L // 2
    tops = {3: inf, 5: -inf, 7: float("nan"), 9: 0.0, 11: 0.0, 13: 1.0, 15: 1e30, 17: -inf, 19: 1e30, 66: inf, 131: 0.0}
    for c, v in tops.items():
        e[:, :, c] = 0
        e[L, :, c] = v
    e[m, :, 20], e[m, :, 22], e[L - 1, :, 24], e[1, :, 26] = inf, float("nan"), -inf, inf
    lm[..., 3] = lm[..., 66] = 1e-30       # products vanish: an infinite state stays infinite
    lm[m, ..., 5] = 0                      # 0 times an infinity from there on
    lm[..., 9] = 1e30                      # products overflow: a state of zero stays zero
    lm[..., 11] = 1e30                     # ... and one that is given a value late does what it does by itself
    e[0, :, 11] = 1.0
    lm[..., 13] = 1e-25
    lm[::2, ..., 15], lm[1::2, ..., 15] = (1e30, 1e-30) if L % 2 == 0 else (1e-30, 1e30)
    lm[..., 19] = lm[..., 15].flip(0) if L % 2 == 0 else 1 / lm[..., 15]       # (the state in between overflows)
    lm[m, ..., 17] = -2.0
    lm[m, ..., 30] = 0
    lm[m:m + 5, ..., 32] = 1.75            # above one
    lm[m, ..., 131] = inf                  # ... and an infinite coefficient
    e[m, :, 131] = 0
    lm[m, ..., 133] = inf
    lm[0, ..., 135] = float("nan")
    e, lm = e.to(st), (lm.to(st) if lam == "token" else lm)
    desc = B.make_desc("rnn", dtype, "tanh", "none", L, N, d, 8, 8, lambda_channel=lam == "channel", lambda_token=lam == "token",
                       loss_every_state=True)
    z = lambda *s: torch.zeros(s, dtype=st, device="cuda")
    p = B.Problem(desc=desc, W1=z(8, d), W2=z(d, 8), U=z(8, 8), lam=lm.cuda(), xin=None, e=e.cuda(),
                  g=torch.full((L + 1, N, d), 5.0, dtype=st, device="cuda"))
    p.workspace = torch.zeros(B.workspace_size(desc), dtype=torch.uint8, device="cuda")
    B.hbp_initial_estimate(p, "auto")
    torch.cuda.synchronize()
    rows = lm.float().numpy()
    with np.errstate(over="ignore", invalid="ignore", under="ignore"):
        want = _walk(e[:L].double().numpy(), [np.broadcast_to(r, (N, d)) for r in rows], e[L].float().numpy())
        want = torch.from_numpy(want).to(st).double().numpy()
    got = p.g.double().cpu().numpy()
    cols = lambda bad: sorted(set(np.argwhere(bad)[:, 2]))
    assert not cols(np.isnan(got) != np.isnan(want)), ("NaN", cols(np.isnan(got) != np.isnan(want)))
    i = np.isinf(want)
    assert not cols((np.isinf(got) != i) | (i & (got != want))), ("infinities", cols((np.isinf(got) != i) | (i & (got != want))))
    f = np.isfinite(want)
    # two roundings to the storage type that may fall apart, and the sums' order over a few states
    got, want = got[f], want[f]
    off = np.abs(got - want) > (2.0 ** -7 if dtype == "bf16" else 1e-5) * (np.abs(want) + 1.0)
    assert not off.any(), (got[off], want[off])
