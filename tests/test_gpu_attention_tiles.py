"""Attention at the edges of its tiling: one tile, odd and even tile counts
(the 64- and the 128-query forward), head counts that are no multiple of eight
(workgroups are numbered heads first) and groups of query heads walked by one
key-tile workgroup, several samples, both head widths.  Element by element
against the oracle, within the bounds derived for the kernels' arithmetic."""
import numpy as np
import pytest
import torch

from oracle import llama_block as lb
from paper_2308_13137_amd import oq
from tests.cases import bf16_exact, dev
from tests.test_gpu_llama import attention_bounds, host

pytestmark = pytest.mark.gpu

CASES = [dict(S=64, ns=3, H=1, Hkv=1), dict(S=320, ns=2, H=5, Hkv=5), dict(S=192, ns=2, H=6, Hkv=2),
         dict(S=384, ns=1, H=3, Hkv=1), dict(S=128, ns=1, H=9, Hkv=9)]


@pytest.mark.parametrize("d", (64, 128))
@pytest.mark.parametrize("c", CASES, ids=[str(c) for c in CASES])
def test_attention_tiles(c, d):
    S, H, Hkv, T = c["S"], c["H"], c["Hkv"], c["S"] * c["ns"]
    rng = np.random.default_rng(31 + S + d + H)
    q, do = (bf16_exact(rng.standard_normal((T, H * d))) for _ in range(2))
    k, v = (bf16_exact(rng.standard_normal((T, Hkv * d)) + rng.standard_normal(Hkv * d))
            for _ in range(2))
    out, P, _ = lb.attention(q, k, v, H, Hkv, d, S, bf16=True)
    ref = (out, *lb.attention_bwd(q, k, v, P, do, H, Hkv, d, S, bf16=True))
    Q, K, V, dO = (dev(x, torch.bfloat16) for x in (q, k, v, do))
    O, lse, _ = oq.attention_fwd(Q, K, V, S, H, Hkv)
    got = (O, *oq.attention_bwd(Q, K, V, dO, lse, S, H, Hkv))
    for name, g, r, b in zip(("O", "dQ", "dK", "dV"), got, ref,
                             attention_bounds(q, k, v, do, H, Hkv, d, S)):
        err = np.abs(host(g).astype(np.float64) - r)
        assert np.all(err <= 2 * b + 1e-30), (name, float(np.max(err / (2 * b + 1e-30))))
