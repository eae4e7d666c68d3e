"""bf16 products with few output tiles (64x64, 128x64 and 128x128 tiles, three
or four K slices in flight) at the edges of the shapes each takes: ragged rows
and columns, as few K slices as stages and fewer, with every epilogue, against
the float64 oracle. Tolerance as for the other bf16 products (one bf16 rounding
of the output, fp32 sums)."""
import math

import numpy as np
import pytest
import torch

from oracle import zsa_oracle as O
from paper_2509_01190_amd import zsa
from tests.helpers import assert_close, dev, f64, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,k", [(801, 768, 64),       # 64x64, one slice (fewer than the stages)
                                   (801, 768, 128),      # two slices
                                   (1025, 784, 192),     # three, ragged rows and columns
                                   (300, 2304, 768),     # 64x64, taken over from the few-row kernel
                                   (70, 16384, 2048),    # 64x64, two per CU
                                   (2049, 768, 3072),    # 128x64
                                   (1537, 1040, 2048),   # 128x64, ragged columns
                                   (3300, 768, 3072),    # 128x128 on 8 waves
                                   (250, 16384, 2048),   # 128x128, one per CU
                                   (1100, 2048, 4160)])  # past the K of the short grids: split where it may
@pytest.mark.parametrize("epi", [zsa.EPI_NONE, zsa.EPI_GELU, zsa.EPI_SWIGLU, zsa.EPI_RESIDUAL, zsa.EPI_ROPE])
@pytest.mark.parametrize("split", [True, False])
def test_linear_short_grids(m, n, k, epi, split):
    hd = 64 if epi == zsa.EPI_ROPE and n % 64 == 0 else 16
    g = np.random.default_rng(m + n + k + epi)
    xd = to_dev(g.standard_normal((m, k)).astype(np.float32), "bf16")
    wd = to_dev((g.standard_normal((n, k)) / math.sqrt(k)).astype(np.float32), "bf16")
    bd = to_dev((0.1 * g.standard_normal(n)).astype(np.float32), "bf16")
    res = to_dev(g.standard_normal((m, n)).astype(np.float32), "bf16") if epi == zsa.EPI_RESIDUAL else None
    pos = g.integers(0, 4096, m).astype(np.int32)
    cols = n // 2 // hd * hd
    kw = dict(residual=res, pos=torch.from_numpy(pos).to(dev()) if epi == zsa.EPI_ROPE else None, head_dim=hd,
              rope_cols=cols, rope_theta=1e4, split=split)
    y = zsa.linear(xd, wd, bd, epi, **kw)
    again = zsa.linear(xd, wd, bd, epi, **kw)
    assert torch.equal(y, again)
    rows = np.unique(np.concatenate([np.arange(33), np.arange(m - 65, m), g.integers(0, m, 64)]))
    rt = torch.from_numpy(rows).to(dev())
    z = f64(xd[rt]) @ f64(wd).T + f64(bd)
    if epi == zsa.EPI_GELU:
        z = O.gelu(z)
    elif epi == zsa.EPI_SWIGLU:
        z = O.silu(z[:, 0::2]) * z[:, 1::2]
    elif epi == zsa.EPI_RESIDUAL:
        z = z + f64(res[rt])
    elif epi == zsa.EPI_ROPE:
        z[:, :cols] = O.rope(z[:, :cols], pos[rows].astype(np.int64), cols // hd, 1e4)
    assert_close(f64(y[rt]), z, 1e-2, f"{m}x{n}x{k} epilogue {epi}")


@pytest.mark.parametrize("m,n,k,hd", [(640, 768, 3104, 0),    # K no multiple of 64, either side of 150 64x64 tiles
                                      (800, 768, 3104, 0),
                                      (100, 6144, 4096, 128),  # rotary heads of 128: few-row
                                      (256, 3072, 1024, 128),  # ... its most rows at this width
                                      (130, 12288, 2112, 128), # ... split K, or 128x128 tiles without the room for it
                                      (512, 6144, 2048, 128)]) # ... 128x128 tiles on most CUs
@pytest.mark.parametrize("split", [True, False])
def test_linear_without_narrow_tiles(m, n, k, hd, split):
    """Products that no 64-wide tile takes."""
    g = np.random.default_rng(m + n + k)
    xd = to_dev(g.standard_normal((m, k)).astype(np.float32), "bf16")
    wd = to_dev((g.standard_normal((n, k)) / math.sqrt(k)).astype(np.float32), "bf16")
    bd = to_dev((0.1 * g.standard_normal(n)).astype(np.float32), "bf16")
    pos = g.integers(0, 4096, m).astype(np.int32)
    cols = n // 2 // hd * hd if hd else 0
    y = zsa.linear(xd, wd, bd, zsa.EPI_ROPE if hd else zsa.EPI_NONE,
                   pos=torch.from_numpy(pos).to(dev()) if hd else None, head_dim=hd, rope_cols=cols, rope_theta=1e4,
                   split=split)
    rows = np.unique(np.concatenate([np.arange(17), np.arange(m - 33, m), g.integers(0, m, 16)]))
    rt = torch.from_numpy(rows).to(dev())
    z = f64(xd[rt]) @ f64(wd).T + f64(bd)
    if hd:
        z[:, :cols] = O.rope(z[:, :cols], pos[rows].astype(np.int64), cols // hd, 1e4)
    assert_close(f64(y[rt]), z, 1e-2, f"{m}x{n}x{k}, rotary heads of {hd}")
