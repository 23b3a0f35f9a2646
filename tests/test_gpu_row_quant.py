"""Row quantisers without LET against the general kernels, bit for bit: s of
ones and zero delta are exact no-ops, so the LET kernels (whose sums run in the
same order) must give the same codes, step sizes, values and gradients at the
edges of the widths the launches choose between.  Type conversion of
unquantised activations against the rounding itself."""
import pytest
import torch

from paper_2308_13137_amd import oq

pytestmark = pytest.mark.gpu

# channels at and just past 1, 2, 3, 4 chunks of 256 threads and 3, 4, 6, 7 of 512
WIDTHS = (64, 2048, 2056, 4096, 6144, 6152, 8192, 8200, 12288, 12296, 16384, 16392, 24576, 24584, 28672, 28680)


def bits_equal(a, b):
    return torch.equal(a.view(torch.int32) if a.dtype == torch.float32 else a,
                       b.view(torch.int32) if b.dtype == torch.float32 else b)


@pytest.mark.parametrize("C", WIDTHS)
@pytest.mark.parametrize("dtype", (torch.float32, torch.bfloat16))
def test_activations_without_let(C, dtype):
    gen = torch.Generator(device="cuda").manual_seed(C)
    T = 5
    X = torch.randn(T, C, generator=gen, device="cuda").to(dtype)
    X[1] = 0                                            # a row without range
    X[2, C // 2] = 40.0
    one, zero = torch.ones(C, device="cuda"), torch.zeros(C, device="cuda")
    other = torch.bfloat16 if dtype == torch.float32 else torch.float32
    for bits in (4, 8):
        plain = oq.act_fakequant_fwd(X, bits, dq_dtype=other)
        let = oq.act_fakequant_fwd(X, bits, s=one, delta=zero, dq_dtype=other)
        assert all(bits_equal(a, b) for a, b in zip(plain, let) if a is not None)
    G = torch.randn(T, C, generator=gen, device="cuda")
    for bits in (4, 16):
        plain = torch.empty_like(G)                     # (no sums wanted: the kernel without LET)
        oq.act_fakequant_bwd_noalloc_into(X, bits, G, plain, None, None)
        let = oq.act_fakequant_bwd(X, bits, G, s=one, delta=zero)[0]
        assert bits_equal(plain, let)
    assert torch.equal(oq.act_fakequant_fwd(X, 16, dq_dtype=other, codes=False, hz=False)[0], X.to(other))


@pytest.mark.parametrize("c_in", WIDTHS[3:])
def test_row_weights_without_let(c_in):
    gen = torch.Generator(device="cuda").manual_seed(c_in)
    n = 7
    W = (0.02 * torch.randn(n, c_in, generator=gen, device="cuda")).bfloat16()
    gl, bl = (torch.full((n, 1), 4.0, device="cuda") for _ in range(2))
    G = torch.randn(n, c_in, generator=gen, device="cuda")
    plain = oq.lwc_fakequant_bwd(W, gl, bl, 4, c_in, G)
    let = oq.lwc_fakequant_bwd(W, gl, bl, 4, c_in, G, s=torch.ones(c_in, device="cuda"), want_d_s=True)
    assert bits_equal(plain[0], let[0]) and bits_equal(plain[1], let[1])
