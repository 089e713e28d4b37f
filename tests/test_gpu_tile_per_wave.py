"""The GEMM of a tile per wave (windows of 9 to 32 rows): bit for bit the rows of windows of up to 8, which another form
computes, on either side of its limits, and within fp32 rounding of the 64-bit product."""
import pytest
import torch

from paper_2404_08698_amd import binding as B

pytestmark = pytest.mark.gpu


# one tile; one per block (rings of 32 k-steps); one or two (257 tiles on 256 compute units); four, and five in fewer blocks; seven per block, and one tile too
# many for that; K of one k-step, of a piece of one, of one and of two buffers, ragged, longer than the ring
@pytest.mark.parametrize("rows", [9, 16, 17, 32])
@pytest.mark.parametrize("n,k", [(16, 32), (48, 8), (512, 992), (512, 1000), (4096, 4104), (4112, 264), (4112, 1000), (8192, 512), (16384, 136), (16400, 136), (28672, 136), (28688, 136), (12288, 4104)])
def test_rows_have_the_bits_of_small_windows(rows, n, k):
    g = torch.Generator(device="cuda").manual_seed(7 * rows + n + k)
    x = torch.empty(rows, k, device="cuda").normal_(generator=g)
    w = torch.empty(n, k, dtype=torch.bfloat16, device="cuda").normal_(0.0, 0.05, generator=g)
    packed = B.pack_weights(w)
    y = B.linear(x, w, B.GEMM_MFMA, packed=packed)
    parts = torch.cat([B.linear(x[r:r + 8].contiguous(), w, B.GEMM_MFMA, packed=packed) for r in range(0, rows, 8)])
    assert torch.equal(y, parts)
    exact = x.double() @ w.double().t()
    # activations as two bf16 terms (2^-17 each), fp32 sums of at most k / 8 + 8 terms in a row
    bound = (2.0 ** -16 + (k / 8 + 8) * 2.0 ** -24) * (x.double().abs() @ w.double().abs().t())
    assert bool(((y.double() - exact).abs() <= bound + 1e-30).all())
