"""Row norms on both sides of the few-row kernel's range: 256 rows and 257,
widths just past its smallest and at its widest, LayerNorm with and without
shift and RMSNorm, both storage types."""
import pytest
import torch

from paper_2509_01190_amd import zsa
from tests.helpers import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [1, 4, 256, 257])
@pytest.mark.parametrize("dtype,d", [(torch.bfloat16, 1032), (torch.bfloat16, 2056), (torch.bfloat16, 8192),
                                     (torch.float32, 516), (torch.float32, 4096)])
@pytest.mark.parametrize("kind,shift", [("layer", True), ("layer", False), ("rms", False)])
def test_norm_rows(rows, dtype, d, kind, shift):
    g = torch.Generator(device=dev()).manual_seed(d + rows)
    x = (torch.randn(rows, d, generator=g, device=dev()) * 3 + 1).to(dtype)
    w = (1 + 0.1 * torch.randn(d, generator=g, device=dev())).to(dtype)
    b = (0.1 * torch.randn(d, generator=g, device=dev())).to(dtype) if shift else None
    y = zsa.norm(x, w, b, zsa.NORM_LAYER if kind == "layer" else zsa.NORM_RMS, 1e-5)
    z = x.double()
    if kind == "layer":
        z = z - z.mean(dim=1, keepdim=True)
    z = z / torch.sqrt((z * z).mean(dim=1, keepdim=True) + 1e-5) * w.double()
    if shift:
        z = z + b.double()
    # one rounding of the result (half a unit of 8 or 24 bits) and, in fp32,
    # those of the row's sums and of the four operations on an element
    lim = 2.0 ** -8 if dtype == torch.bfloat16 else 8 * 2.0 ** -24
    assert ((y.double() - z).norm() / z.norm()).item() <= lim
