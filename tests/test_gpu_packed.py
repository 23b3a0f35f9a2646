"""Parity of the deployment kernels (Sec. 4.5) with the oracle: the packed code
layout bit for bit, and the weight-only quantised linear element by element
within a bound derived from its fp32 arithmetic.

Bound of the linear.  The vector kernel (one or two tokens in groups that are no
multiple of 128) forms, per run of 32 codes, p = sum x (128 + q)
with bf16 x and exact bf16 codes (every product exact in fp32), then
h * (p - (128 + z) * xs) with xs = sum x, and sums runs and lanes in fp32.  Each
of the at most ~40 roundings on the way contributes at most 2^-24 times a
partial sum bounded by sum_c |x_c| (256 + q_c + |z_g|) h_g, so
|Y - Y_oracle| <= 4e-6 * sum_c |x_c| (256 + q_c + |z_g|) h_g, plus half a bf16
ulp of |Y| when Y is stored in bf16.

Everything else runs on matrix cores, with the offset 2^bits instead of 128: each
128-channel block's p is a chain of four 32-term matrix products, up to 128 fp32
roundings of a partial sum bounded by the same magnitude, plus the ~40 of the
rest: (128 + 40) 2^-24 ~ 1.0e-5 times the same sum.  The matrix instructions
round far less often than once per term (the largest error measured is 0.01 of
the vector kernel's bound), so only 8 or more tokens in groups of 128 are given
that bound and all others the vector kernel's."""
import numpy as np
import pytest
import torch

from oracle.packed import pack_codes as o_pack
from oracle.packed import packed_linear as o_linear
from oracle.quant import bf16_round
from paper_2308_13137_amd import oq

pytestmark = pytest.mark.gpu
DEV = "cuda"


def make_linear(seed, bits, n_tok, c_out, c_in, group, bias, z_spread=0):
    rng = np.random.default_rng(seed)
    q = rng.integers(0, 2 ** bits, size=(c_out, c_in), dtype=np.uint8)
    ng = c_in // group
    h = rng.uniform(1e-3, 2e-2, size=(c_out, ng)).astype(np.float32)
    z = rng.integers(-z_spread, 2 ** bits + z_spread, size=(c_out, ng)).astype(np.float32)
    X = rng.standard_normal((n_tok, c_in)).astype(np.float32)
    heavy = rng.choice(c_in, size=max(1, c_in // 100), replace=False)
    X[:, heavy] *= 10.0                               # a few outlier channels
    X = bf16_round(X)
    B = rng.standard_normal(c_out).astype(np.float32) if bias else None
    return q, h, z, X, B


def mfma_path(n_tok, group):
    """The cases that are given the matrix cores' bound."""
    return n_tok >= 8 and group == 128


def bound(q, h, z, X, group):
    mag = (256.0 + q.astype(np.float64) + np.repeat(np.abs(z), group, axis=1)) * np.repeat(h, group, axis=1)
    eps = (128 + 40) * 2.0 ** -24 if mfma_path(X.shape[0], group) else 4e-6
    return eps * (np.abs(X).astype(np.float64) @ mag.T)


def to_dev(a, dtype=None):
    t = torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
    return t if dtype is None else t.to(dtype)


@pytest.mark.parametrize("bits,c_out,c_in", [
    (2, 3, 32), (3, 5, 96), (4, 64, 4096), (5, 7, 160), (6, 33, 224), (7, 2, 32), (8, 17, 256),
    (3, 129, 11008), (2, 0, 64),
])
def test_pack_codes_bit_exact(bits, c_out, c_in):
    rng = np.random.default_rng(bits * 1000 + c_in)
    codes = rng.integers(0, 2 ** bits, size=(c_out, c_in), dtype=np.uint8)
    got = oq.pack_codes(to_dev(codes), bits).cpu().numpy()
    assert got.shape == (c_out, c_in * bits // 8)
    assert np.array_equal(got, o_pack(codes, bits))


LINEAR = [
    # bits, n_tok, c_out, c_in, group, bias, out dtype, z outside [0, qmax]
    (4, 1, 4096, 4096, 128, False, torch.float32, 0),     # 7B q/k/v/o shape
    (4, 1, 1000, 11008, 128, True, torch.float32, 0),     # down_proj width, ragged rows
    (4, 2, 12289, 1024, 128, True, torch.float32, 0),     # more row tiles than resident workgroups
    (3, 1, 333, 4096, 128, False, torch.float32, 0),
    (2, 1, 257, 4096, 64, False, torch.float32, 0),
    (4, 3, 129, 512, 32, True, torch.bfloat16, 2),
    (4, 8, 100, 4096, 128, False, torch.float32, 0),
    (4, 13, 50, 1024, 1024, True, torch.float32, 0),      # one group per row
    (2, 8, 64, 11008, 128, False, torch.float32, 0),
    (5, 2, 40, 96, 32, False, torch.float32, 3),
    (6, 5, 40, 160, 32, True, torch.float32, 0),
    (7, 4, 17, 224, 32, False, torch.bfloat16, 0),
    (3, 6, 1, 32, 32, True, torch.float32, 1),
    # groups of a number of runs that is not a power of two (3 and 344 runs)
    (4, 2, 70, 288, 96, True, torch.float32, 0),
    (3, 1, 33, 11008, 11008, False, torch.float32, 0),
    # the widest input: past what LDS keeps of 3 tokens
    (4, 3, 7, 65536, 128, False, torch.float32, 0),
    # groups of 128: 16-, 24- and 32-token launches, 70 = 32 + 32 + 6 tokens,
    # ragged rows, the 7B shapes, every code width
    (4, 16, 4096, 4096, 128, True, torch.float32, 0),
    (4, 64, 1000, 11008, 128, False, torch.float32, 0),
    (3, 33, 129, 11008, 128, True, torch.bfloat16, 1),
    (2, 70, 300, 4096, 128, False, torch.float32, 0),
    (5, 20, 17, 256, 128, True, torch.float32, 2),
    (6, 9, 40, 384, 128, False, torch.float32, 0),
    (7, 24, 33, 128, 128, True, torch.float32, 0),
    # wide inputs in launches of 32 + 8 and of 20 tokens
    (4, 40, 7, 32768, 128, True, torch.float32, 0),
    (3, 20, 5, 65536, 128, False, torch.bfloat16, 0),
    # more 16-row tiles than CUs (8, 12 and 40 tokens)
    (4, 8, 4200, 1024, 128, False, torch.float32, 0),
    (5, 12, 4113, 512, 128, True, torch.bfloat16, 1),
    (4, 40, 4352, 640, 128, True, torch.float32, 0),
    # two 16-row tiles per workgroup (ragged last one)
    (4, 12, 16400, 512, 128, True, torch.bfloat16, 0),
    (3, 40, 16384, 1024, 128, False, torch.float32, 1),
    (5, 8, 16424, 384, 128, True, torch.float32, 0),
    (4, 24, 9000, 256, 128, True, torch.float32, 0),      # from 8,192 rows at 17-24 tokens
    (2, 20, 16400, 256, 128, False, torch.bfloat16, 1),
    (6, 8, 16390, 128, 128, True, torch.float32, 0),
    (7, 33, 16384, 384, 128, False, torch.float32, 0),
]


@pytest.mark.parametrize("case", LINEAR, ids=[f"b{c[0]}_t{c[1]}_{c[2]}x{c[3]}_g{c[4]}" for c in LINEAR])
def test_packed_linear_matches_oracle(case):
    bits, n_tok, c_out, c_in, group, bias, odt, zs = case
    q, h, z, X, B = make_linear(100 + LINEAR.index(case), bits, n_tok, c_out, c_in, group, bias, zs)
    P = o_pack(q, bits)
    ref = o_linear(X, P, bits, group, h, z, B)
    Y = oq.packed_linear(to_dev(X, torch.bfloat16), to_dev(P), bits, group, to_dev(h), to_dev(z),
                         None if B is None else to_dev(B), out_dtype=odt)
    torch.cuda.synchronize()
    got = Y.float().cpu().numpy().astype(np.float64)
    tol = bound(q, h, z, X, group)
    if odt == torch.bfloat16:
        tol = tol + np.abs(ref) * 2.0 ** -8
    err = np.abs(got - ref)
    assert np.all(err <= tol), (err.max(), (err / tol).max())


def test_packed_linear_empty_and_reproducible():
    q, h, z, X, _ = make_linear(9, 4, 5, 300, 4096, 128, False)
    Xd, Pd, hd, zd = to_dev(X, torch.bfloat16), to_dev(o_pack(q, 4)), to_dev(h), to_dev(z)
    assert oq.packed_linear(Xd[:0], Pd, 4, 128, hd, zd).shape == (0, 300)
    a = oq.packed_linear(Xd, Pd, 4, 128, hd, zd)
    b = oq.packed_linear(Xd, Pd, 4, 128, hd, zd)
    torch.cuda.synchronize()
    assert torch.equal(a, b)
    # one token at a time gives the same bits as the batch (fixed sum order)
    for t in range(5):
        assert torch.equal(oq.packed_linear(Xd[t:t + 1], Pd, 4, 128, hd, zd)[0], a[t])


@pytest.mark.parametrize("c_out", [260, 9000, 16400])
def test_matrix_core_batches_give_each_token_the_same_bits(c_out):
    """On matrix cores a token's outputs depend only on its own column: a
    token gives the same bits in batches of 8, 20 and 64.  Many rows (16,384;
    12,288 in launches of 5-16 tokens, 8,192 of 17-24) make a workgroup take two
    16-row tiles; its rows give the same bits as the same rows in a launch of
    one tile per workgroup."""
    q, h, z, X, B = make_linear(12, 4, 64, c_out, 4096, 128, True)
    Xd, Pd, hd, zd, Bd = (to_dev(X, torch.bfloat16), to_dev(o_pack(q, 4)), to_dev(h), to_dev(z),
                          to_dev(B))
    full = oq.packed_linear(Xd, Pd, 4, 128, hd, zd, Bd)
    a = oq.packed_linear(Xd[:8], Pd, 4, 128, hd, zd, Bd)
    b = oq.packed_linear(Xd[30:50], Pd, 4, 128, hd, zd, Bd)
    torch.cuda.synchronize()
    assert torch.equal(a, full[:8])
    assert torch.equal(b, full[30:50])
    if c_out > 260:
        head = oq.packed_linear(Xd, Pd[:260], 4, 128, hd[:260], zd[:260], Bd[:260])
        torch.cuda.synchronize()
        assert torch.equal(head, full[:, :260])


def test_gate_up_stack_full_size_sampled_rows():
    # 7B gate and up projections stacked (22016 x 4096), 4-bit g128, one token:
    # every row is independent, so sampled rows are checked against the oracle
    bits, c_out, c_in, group = 4, 22016, 4096, 128
    q, h, z, X, B = make_linear(21, bits, 1, c_out, c_in, group, True)
    P = o_pack(q, bits)
    Y = oq.packed_linear(to_dev(X, torch.bfloat16), to_dev(P), bits, group, to_dev(h), to_dev(z),
                         to_dev(B)).cpu().numpy().astype(np.float64)
    rows = np.random.default_rng(0).choice(c_out, size=64, replace=False)
    rows = np.concatenate([rows, [0, c_out - 1]])
    ref = o_linear(X, P[rows], bits, group, h[rows], z[rows], B[rows])
    tol = bound(q[rows], h[rows], z[rows], X, group)
    assert np.all(np.abs(Y[:, rows] - ref) <= tol)


def test_pack_and_linear_agree_with_lwc_dequantised_weight():
    # codes, h, z of the library's own Eq.2 forward, packed by the library: the
    # packed linear reproduces X W_dq^T with W_dq that forward's fp32 output
    rng = np.random.default_rng(4)
    c_out, c_in, group, bits = 96, 1024, 128, 3
    W = to_dev((0.02 * rng.standard_normal((c_out, c_in))).astype(np.float32), torch.bfloat16)
    gl = torch.full((c_out, c_in // group), 2.0, device=DEV)
    Wdq, codes, h, z = oq.lwc_fakequant_fwd(W, gl, gl, bits, group, dq_dtype=torch.float32)
    X = to_dev(bf16_round(rng.standard_normal((2, c_in)).astype(np.float32)), torch.bfloat16)
    Y = oq.packed_linear(X, oq.pack_codes(codes, bits), bits, group, h, z)
    ref = X.double() @ Wdq.double().T
    torch.cuda.synchronize()
    zz = z.abs().repeat_interleave(group, 1).double()
    hh = h.repeat_interleave(group, 1).double()
    scale = X.double().abs() @ ((256 + codes.double() + zz) * hh).T
    assert torch.all((Y.double() - ref).abs() <= 4e-6 * scale)


@pytest.mark.parametrize("n_tok,group", [(2, 128), (12, 128), (24, 128), (2, 64)])
def test_packed_linear_graph_replays_match_eager(n_tok, group):
    # a decode loop replays the same launches from a HIP graph: every replay,
    # with eager work and new activations between replays, matches eager runs
    # (2 tokens in groups of 64: the vector kernel; the others: matrix cores)
    q, h, z, X, B = make_linear(31, 4, n_tok, 700, 4096, group, True)
    Xd, Pd, hd, zd, Bd = (to_dev(X, torch.bfloat16), to_dev(o_pack(q, 4)), to_dev(h), to_dev(z),
                          to_dev(B))
    Y = torch.empty((n_tok, 700), device=DEV)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        oq.packed_linear_into(Xd, Pd, 4, group, hd, zd, Y, B=Bd)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        oq.packed_linear_into(Xd, Pd, 4, group, hd, zd, Y, B=Bd)
    rng = np.random.default_rng(32)
    for i in range(4):
        if i:
            Xd.copy_(to_dev(bf16_round(rng.standard_normal((n_tok, 4096)).astype(np.float32)),
                            torch.bfloat16))
        want = oq.packed_linear(Xd, Pd, 4, group, hd, zd, Bd)
        Y.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(Y, want), i


@pytest.mark.parametrize("let", [False, True], ids=["w3_g64", "w4_let"])
def test_block_export_matches_oracle(let):
    """Algorithm 1's quantised block: every linear's packed codes, h and z equal
    the oracle's Eq. 2 quantisation of s (.) W bit for bit, and the folded bias
    is the oracle's B + delta W."""
    from oracle.let import let_bias
    from oracle.quant import lwc_fwd as o_lwc
    from tests.cases import make_problem, small_llama
    if let:
        w = small_llama("export_let", hidden=256, ffn=512, T=128, w_bits=4, let=True, act_bits=4)
    else:
        w = small_llama("export", hidden=256, ffn=512, T=128, w_bits=3, group=64)
    P = make_problem(w, seed=3, logit="random", bias=True)
    blk = oq.Block(w.T, [(s.width, s.let, s.act_bits) for s in w.sites],
                   [(l.site, l.c_out, l.bits, l.group) for l in w.linears], dtype=torch.bfloat16)
    opt = lambda xs: [None if x is None else to_dev(x) for x in xs]
    outs = blk.export([to_dev(x, torch.bfloat16) for x in P["W"]], opt(P["gamma_logit"]),
                      opt(P["beta_logit"]), s=opt(P["s"]), delta=opt(P["delta"]), B=opt(P["B"]))
    torch.cuda.synchronize()
    for l, lin in enumerate(w.linears):
        site = w.sites[lin.site]
        st = o_lwc(P["W"][l], P["gamma_logit"][l], P["beta_logit"][l], lin.bits, lin.group,
                   s=P["s"][lin.site] if site.let else None)
        packed, h, z, bt = (t.cpu().numpy() for t in outs[l])
        assert np.array_equal(packed, o_pack(st["codes"], lin.bits)), l
        assert np.array_equal(h, st["h_g"]) and np.array_equal(z, st["z_g"]), l
        want = let_bias(P["W"][l], P["B"][l], P["delta"][lin.site]) if site.let else P["B"][l]
        scale = np.abs(P["W"][l]).astype(np.float64) @ (np.abs(P["delta"][lin.site]) if site.let
                                                        else np.zeros(site.width)) + np.abs(want)
        assert np.all(np.abs(bt - want) <= 1e-5 * scale + 1e-30), l
