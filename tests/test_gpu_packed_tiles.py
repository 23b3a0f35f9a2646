"""Packed linear: the edges of its kernels' tiles, against the oracle.

Up to 96 tokens go in launches of at most 32 (4 tokens kept in LDS, 8, 16, 24 or 32
staged per block), more through the tiled kernel (64 tokens x 128 outputs).
Blocks of 128 channels hold one, two or four parts by the group size; inputs
that are no multiple of 128 channels take dword copies and a short last block.
The tolerance is the one derived for the packed linear: exact products, every
rounding at most 2^-24 of a partial sum bounded by sum |x| (256 + q + |z|) h.
"""
import numpy as np
import pytest
import torch

from oracle.packed import pack_codes as o_pack, packed_linear as o_linear
from paper_2308_13137_amd import oq
from tests.test_gpu_packed import bound, make_linear, to_dev

pytestmark = pytest.mark.gpu

CASES = [
    # bits, n_tok, c_out, c_in, group, bias, out dtype
    (4, 97, 129, 256, 128, True, torch.float32),       # first tiled size, ragged both ways
    (4, 128, 128, 384, 128, False, torch.bfloat16),    # whole tiles, odd number of blocks
    (3, 130, 257, 640, 64, True, torch.float32),       # two parts per block
    (2, 100, 40, 288, 96, False, torch.float32),       # 32-channel parts, short last block
    (5, 193, 33, 160, 32, True, torch.bfloat16),
    (6, 97, 130, 4096, 4096, False, torch.float32),    # one group per row
    (7, 111, 1, 32, 32, True, torch.float32),
    (4, 4, 17, 96, 32, True, torch.float32),           # dword copies, K shorter than the waves
    (2, 3, 50, 2080, 32, False, torch.float32),        # 65 runs: short last block
    (3, 16, 31, 2080, 160, True, torch.float32),
    (7, 32, 33, 1056, 96, True, torch.bfloat16),       # wide codes: 32 tokens as 24 + 8
    (4, 32, 48, 1152, 64, True, torch.float32),        # one launch of 32, two parts
    (2, 31, 17, 2304, 128, False, torch.float32),
    (6, 17, 40, 512, 256, False, torch.float32),       # groups of two blocks
    (2, 4, 4112, 1280, 64, True, torch.float32),       # two row tiles, ragged last one
    (4, 2, 16400, 256, 128, True, torch.float32),
    (5, 5, 12304, 384, 32, False, torch.float32),
    (4, 4, 70, 22016, 128, False, torch.float32),      # 4 tokens past what LDS keeps
    (5, 6, 40, 640, 64, True, torch.float32),          # rings of 8 tokens, two parts
    (7, 8, 33, 1056, 32, False, torch.bfloat16),       # and by dword copies
    (4, 5, 13320, 256, 128, True, torch.float32),      # and two row tiles
    (4, 27, 5130, 384, 128, True, torch.float32),      # codes through registers: ragged rows and tokens, odd block count
    (3, 32, 5121, 128, 128, False, torch.bfloat16),    # one block: seven waves without one
    (2, 25, 5152, 2304, 768, False, torch.float32),
    (7, 32, 33, 1152, 128, True, torch.float32),       # one row tile at wide codes
    (6, 29, 5136, 512, 256, False, torch.bfloat16),
    (6, 45, 64, 384, 128, True, torch.float32),        # 24 + 21 tokens
]


@pytest.mark.parametrize("case", CASES, ids=[f"b{c[0]}_t{c[1]}_{c[2]}x{c[3]}_g{c[4]}" for c in CASES])
def test_packed_linear_tile_edges(case):
    bits, n_tok, c_out, c_in, group, bias, odt = case
    q, h, z, X, B = make_linear(900 + CASES.index(case), bits, n_tok, c_out, c_in, group, bias, 0)
    P = o_pack(q, bits)
    ref = o_linear(X, P, bits, group, h, z, B)
    Y = oq.packed_linear(to_dev(X, torch.bfloat16), to_dev(P), bits, group, to_dev(h), to_dev(z),
                         None if B is None else to_dev(B), out_dtype=odt)
    torch.cuda.synchronize()
    tol = bound(q, h, z, X, group)
    if odt == torch.bfloat16:
        tol = tol + np.abs(ref) * 2.0 ** -8
    assert np.all(np.abs(Y.float().cpu().numpy().astype(np.float64) - ref) <= tol)


# One or two tokens in groups that are no multiple of 128: the vector kernel.  A
# wave takes row pairs in turn and each in blocks of 4096 channels, the next block
# loading while one computes: a second, partial block, more row pairs than the
# device's waves hold at once (8 per CU and SIMD at most: 16384 rows), and both.
VECTOR = [
    # bits, n_tok, c_out, c_in, group, bias, out dtype
    (2, 1, 100, 11008, 64, False, torch.float32),      # three blocks, the last partial
    (4, 2, 33, 11008, 64, True, torch.float32),
    (3, 2, 41, 4128, 96, False, torch.bfloat16),       # one run past a block; 43 groups of 3 runs
    (4, 1, 7, 8192, 32, True, torch.float32),          # two whole blocks
    (3, 1, 40001, 160, 32, True, torch.float32),       # several row pairs a wave, odd count
    (2, 2, 40001, 192, 96, False, torch.float32),
    (4, 1, 33001, 4160, 64, True, torch.float32),      # both
    (5, 2, 33001, 4128, 32, True, torch.bfloat16),
]


@pytest.mark.parametrize("case", VECTOR, ids=[f"b{c[0]}_t{c[1]}_{c[2]}x{c[3]}_g{c[4]}" for c in VECTOR])
def test_vector_kernel_walks(case):
    bits, n_tok, c_out, c_in, group, bias, odt = case
    q, h, z, X, B = make_linear(500 + VECTOR.index(case), bits, n_tok, c_out, c_in, group, bias, 0)
    P = o_pack(q, bits)
    Y = oq.packed_linear(to_dev(X, torch.bfloat16), to_dev(P), bits, group, to_dev(h), to_dev(z),
                         None if B is None else to_dev(B), out_dtype=odt)
    got = Y.float().cpu().numpy().astype(np.float64)
    # every row where they are few, else every 97th and the first and last ones
    rows = np.unique(np.r_[0:64, 0:c_out:97, c_out - 64:c_out]) if c_out > 1000 else np.arange(c_out)
    ref = o_linear(X, P[rows], bits, group, h[rows], z[rows], None if B is None else B[rows])
    tol = bound(q[rows], h[rows], z[rows], X, group)
    if odt == torch.bfloat16:
        tol = tol + np.abs(ref) * 2.0 ** -8
    assert np.all(np.abs(got[:, rows] - ref) <= tol)


# bits, c_in, group (uneven shares of K, fewer super-blocks than waves, an odd
# number of blocks among them)
SAME = [(4, 4096, 128), (3, 11008, 128), (2, 128, 128), (7, 384, 384), (6, 5120, 5120), (4, 1152, 128),
        (5, 3328, 256), (3, 22016, 128)]


def check_batches(case, c_out, sizes):
    bits, c_in, group = case
    most = sizes[-1]
    q, h, z, X, B = make_linear(7, bits, most, c_out, c_in, group, True, 0)
    Xd, Pd, hd, zd, Bd = to_dev(X, torch.bfloat16), to_dev(o_pack(q, bits)), to_dev(h), to_dev(z), to_dev(B)
    full = oq.packed_linear(Xd, Pd, bits, group, hd, zd, Bd)
    for n in sizes[:-1]:
        for lo in {0, most - n}:
            part = oq.packed_linear(Xd[lo:lo + n], Pd, bits, group, hd, zd, Bd)
            assert torch.equal(part, full[lo:lo + n]), (n, lo)


@pytest.mark.parametrize("c_out", [70, 5130, 16400])
@pytest.mark.parametrize("case", SAME, ids=[f"b{c[0]}_{c[1]}_g{c[2]}" for c in SAME])
def test_a_tokens_outputs_do_not_depend_on_its_batch(case, c_out):
    """Groups that are a multiple of 128: kept activations (to 4 tokens), rings of
    8, 16, 24 and 32 tokens, codes through registers (25 to 32 tokens of 5130 rows
    or at 6 and 7 bits), several launches, one and two row tiles, whole and ragged
    token tiles sum every product over K in the same order."""
    if c_out > 6000 and case[1] > 6000:
        c_out = 8200
    check_batches(case, c_out, (1, 2, 3, 4, 5, 8, 16, 17, 24, 25, 32, 33, 40, 96, 97, 128, 200))


@pytest.mark.parametrize("sizes", [(1, 2), (3, 4, 5, 16, 17, 32, 40, 96), (97, 128, 200)],
                         ids=["vector", "small", "tiled"])
@pytest.mark.parametrize("case", [(2, 5120, 64), (5, 2080, 32), (4, 288, 96)],
                         ids=["g64", "g32_dword", "g96_dword"])
def test_other_groups_do_not_depend_on_the_batch_within_a_kernel(case, sizes):
    check_batches(case, 70, sizes)


def test_a_row_of_nan_steps_leaves_the_others_alone():
    # reads past a row's end (short last block) meet the next row's step size
    q, h, z, X, _ = make_linear(77, 4, 3, 20, 160, 32, False, 0)
    h2 = h.copy()
    h2[7] = np.nan
    a, b = (oq.packed_linear(to_dev(X, torch.bfloat16), to_dev(o_pack(q, 4)), 4, 32, to_dev(v), to_dev(z))
            for v in (h, h2))
    torch.cuda.synchronize()
    keep = [o for o in range(20) if o != 7]
    assert torch.equal(a[:, keep], b[:, keep]) and torch.isnan(b[:, 7]).all()
