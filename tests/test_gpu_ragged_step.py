"""The calibration step at token and row counts that are no multiple of 64: the
gradient products pad their K with zeros in the workspace, and a weight-only
site's product re-reads the last row of the caller's X.  Bounds of the block
step: normwise 1e-3, per element 1e-2 of the value or of 1e-2 of the largest."""
import numpy as np
import pytest
import torch

from oracle.block import block_step
from paper_2308_13137_amd import oq
from tests.cases import dev, make_problem, normwise, small_llama

pytestmark = pytest.mark.gpu

CASES = [  # tokens, hidden, ffn, kv rows, bits, group, LET, activation bits, K splits of the weight gradient
    (8, 128, 256, 128, 4, 64, False, 16, 1),     # less than one stage
    (72, 128, 256, 72, 3, 128, False, 16, 1),    # one stage and 8 rows
    (120, 256, 512, 200, 4, None, True, 4, 1),   # ragged stacked rows too
    (1016, 256, 512, 256, 2, 64, False, 16, 1),
    (4104, 256, 512, 256, 4, None, True, 16, 1),  # 65 stages: no split
    (2040, 256, 768, 8, 4, 32, False, 16, 2),
    (4088, 256, 512, 200, 4, None, True, 4, 4),  # ragged rows and tokens, parts summed by the LET backward
    (2040, 256, 512, 256, 4, None, True, 16, 2),
]


@pytest.mark.parametrize("case", CASES, ids=[f"t{c[0]}_h{c[1]}_kv{c[3]}_g{c[5]}{'_let' if c[6] else ''}" for c in CASES])
def test_ragged_step_matches_oracle(case):
    T, hidden, ffn, kv, bits, group, let, act, splits = case
    w = small_llama("ragged", hidden=hidden, ffn=ffn, T=T, w_bits=bits, group=group, kv=kv, let=let, act_bits=act)
    P = make_problem(w, seed=5, logit="random")
    dt = torch.bfloat16
    blk = oq.Block(T, [(s.width, s.let, s.act_bits) for s in w.sites],
                   [(l.site, l.c_out, l.bits, l.group) for l in w.linears], dtype=dt)
    assert all(p["direct"] and p["wgrad_splits"] == splits for p in blk.plan())
    blk.ws.fill_(0xFF)                            # NaN everywhere a pad is forgotten
    opt = lambda xs: [None if x is None else dev(x) for x in xs]
    # X ends where its allocation's tokens do: the rows after it are NaN
    Xp = [torch.full((T + 64, s.width), float("nan"), dtype=dt, device="cuda") for s in w.sites]
    for x, v in zip(Xp, P["X"]):
        x[:T] = dev(v, dt)
    loss = blk.step([x[:T] for x in Xp], [dev(np.ascontiguousarray(y.T), dt) for y in P["Y"]],
                    [dev(x, dt) for x in P["W"]], opt(P["gamma_logit"]), opt(P["beta_logit"]),
                    s=opt(P["s"]), delta=opt(P["delta"]))
    torch.cuda.synchronize()
    params = {k: P[k] for k in ("W", "B", "gamma_logit", "beta_logit", "s", "delta")}
    ref_loss, ref = block_step(w.oracle_desc(), P["X"], P["Y"], params)
    assert abs(float(loss) - ref_loss) <= 1e-3 * abs(ref_loss)
    pairs = [(g, r) for got, name in ((blk.d_gamma, "d_gamma_logit"), (blk.d_beta, "d_beta_logit"))
             for g, r in zip(got, ref[name])]
    if let and act < 16:                          # (without it the LET gradients nearly cancel)
        pairs += [(g, r) for got, name in ((blk.d_s, "d_s"), (blk.d_delta, "d_delta"))
                  for g, r in zip(got, ref[name]) if g is not None]
    for g, r in pairs:
        g = g.cpu().numpy().astype(np.float64)
        assert normwise(g, r) <= 1e-3
        assert np.all(np.abs(g - r) <= 1e-2 * np.maximum(np.abs(r), 1e-2 * np.abs(r).max()))


FP32 = [  # tokens, hidden, ffn, bits, group, LET, activation bits
    (8, 64, 128, 4, 64, False, 16),              # less than one 16 x 16 tile of tokens
    (72, 128, 192, 3, 64, True, 4),              # operands read as stored, every orientation
    (264, 136, 264, 4, 8, True, 16),             # K = 136: a short last stretch of 64
    (1032, 512, 1024, 2, 64, True, 4),           # 64 x 64 tiles in the gate/up product, wave tiles elsewhere
]


@pytest.mark.parametrize("case", FP32, ids=[f"t{c[0]}_h{c[1]}{'_let' if c[5] else ''}" for c in FP32])
def test_fp32_step_matches_oracle(case):
    """fp32 workloads: products of few tiles on wave tiles, others on 64 x 64;
    1e-4 normwise and 1e-3 per element, as the fp32 block step's bounds."""
    from dataclasses import replace
    T, hidden, ffn, bits, group, let, act = case
    w = replace(small_llama("fp32", hidden=hidden, ffn=ffn, T=T, w_bits=bits, group=group, let=let, act_bits=act),
                bf16=False)
    P = make_problem(w, seed=6, logit="random")
    blk = oq.Block(T, [(s.width, s.let, s.act_bits) for s in w.sites],
                   [(l.site, l.c_out, l.bits, l.group) for l in w.linears], dtype=torch.float32)
    blk.ws.fill_(0xFF)
    opt = lambda xs: [None if x is None else dev(x) for x in xs]
    loss = blk.step(opt(P["X"]), [dev(np.ascontiguousarray(y.T)) for y in P["Y"]], opt(P["W"]),
                    opt(P["gamma_logit"]), opt(P["beta_logit"]), s=opt(P["s"]), delta=opt(P["delta"]))
    torch.cuda.synchronize()
    params = {k: P[k] for k in ("W", "B", "gamma_logit", "beta_logit", "s", "delta")}
    ref_loss, ref = block_step(w.oracle_desc(), P["X"], P["Y"], params)
    assert abs(float(loss) - ref_loss) <= 1e-4 * abs(ref_loss)
    names = [(blk.d_gamma, "d_gamma_logit"), (blk.d_beta, "d_beta_logit")]
    if act < 16:
        names += [(blk.d_s, "d_s"), (blk.d_delta, "d_delta")]
    for got, name in names:
        for g, r in zip(got, ref[name]):
            if g is None:
                continue
            g = g.cpu().numpy().astype(np.float64)
            assert normwise(g, r) <= 1e-4, name
            assert np.all(np.abs(g - r) <= 1e-3 * np.maximum(np.abs(r), 1e-2 * np.abs(r).max())), name
