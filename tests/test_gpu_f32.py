"""The fp32 matrix-instruction kernels (projections, attention, scores) at
the edges of their tiles, against the float64 oracle. Tolerances are those of
the other fp32 kernel tests: 2e-5 for sums over K (fp32 accumulation), 1e-5
for attention, 1e-4 for scores (exp2 of an fp32 exponent)."""
import math

import numpy as np
import pytest
import torch

from oracle import zsa_oracle as O
from paper_2509_01190_amd import zsa
from tests.helpers import assert_close, dev, f64, score_err, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,k,hd", [(1, 16, 4, 16),           # one output block, one wave's range
                                      (33, 48, 132, 16),        # ragged blocks, K tail of 4
                                      (65, 128, 1000, 32),      # every wave a range, rotary pair in 32 columns
                                      (1030, 1040, 68, 16),     # 64 x 64 tiles, K not a whole slice
                                      (700, 768, 96, 64),       # rotary heads of 64: 64 x 64 tiles
                                      (2100, 4112, 36, 16),     # 128 x 128 tiles, ragged
                                      (130, 256, 40, 128),      # rotary heads of 128: 64 x 128 tiles
                                      (4200, 2176, 36, 128)])   # ... 128 x 128 tiles
@pytest.mark.parametrize("epi", [zsa.EPI_NONE, zsa.EPI_GELU, zsa.EPI_SWIGLU, zsa.EPI_RESIDUAL, zsa.EPI_ROPE])
def test_linear_f32_tiles(m, n, k, hd, epi):
    g = np.random.default_rng(m + n + k + epi)
    xd = to_dev(g.standard_normal((m, k)).astype(np.float32), "f32")
    wd = to_dev((g.standard_normal((n, k)) / math.sqrt(k)).astype(np.float32), "f32")
    bd = to_dev((0.1 * g.standard_normal(n)).astype(np.float32), "f32")
    res = to_dev(g.standard_normal((m, n)).astype(np.float32), "f32") if epi == zsa.EPI_RESIDUAL else None
    pos = g.integers(0, 4096, m).astype(np.int32)
    cols = n // hd * hd
    y = zsa.linear(xd, wd, bd, epi, residual=res, pos=torch.from_numpy(pos).to(dev()) if epi == zsa.EPI_ROPE else None,
                   head_dim=hd, rope_cols=cols, rope_theta=1e4)
    z = f64(xd) @ f64(wd).T + f64(bd)
    if epi == zsa.EPI_GELU:
        z = O.gelu(z)
    elif epi == zsa.EPI_SWIGLU:
        z = O.silu(z[:, 0::2]) * z[:, 1::2]
    elif epi == zsa.EPI_RESIDUAL:
        z = f64(res) + z
    elif epi == zsa.EPI_ROPE:
        z[:, :cols] = O.rope(z[:, :cols], pos.astype(np.int64), cols // hd, 1e4)
    assert_close(f64(y), z, 2e-5, f"fp32 product {m}x{n}x{k} epilogue {epi}")


@pytest.mark.parametrize("dtype,hd", [("f32", 16), ("f32", 32), ("f32", 64), ("f32", 128), ("bf16", 16)])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("hkv", [4, 2])
def test_attention_f32_tile_edges(dtype, hd, causal, hkv):
    """Sequences of 0 to 300 rows: under, at and past one 32-row tile, and past
    one round of the four waves."""
    lens, H = [0, 1, 31, 32, 33, 128, 129, 300], 4
    g = np.random.default_rng(hd + hkv + causal)
    T, d, kvd = sum(lens), H * hd, hkv * hd
    t = to_dev(g.standard_normal((T, d + 2 * kvd)).astype(np.float32) * np.float32(1.5), dtype)
    q, k, v = t.split([d, kvd, kvd], dim=1)
    seqs = zsa.Seqs(lens, dev())
    out, lse, scores = zsa.attention_with_scores(q, k, v, H, seqs, causal, n_kv_heads=hkv)
    q64, k64, v64 = (f64(a) for a in (q, k, v))
    k64, v64 = (np.repeat(a.reshape(T, hkv, hd), H // hkv, axis=1).reshape(T, d) for a in (k64, v64))
    for b, n in enumerate(lens):
        if n == 0:
            continue
        s = slice(int(seqs.host[b]), int(seqs.host[b + 1]))
        o, l, sc = O.attention(q64[s], k64[s], v64[s], np.arange(n), H, causal)
        assert_close(f64(out)[s], o, 1e-2 if dtype == "bf16" else 1e-5, f"attention, {n} rows")
        assert_close(f64(lse)[:, s], l, 1e-5, f"log-sum-exp, {n} rows")
        assert score_err(f64(scores)[s], sc) <= 1e-4


@pytest.mark.parametrize("bad", [math.inf, -math.inf, math.nan])
def test_attention_f32_masked_rows_stay_out(bad):
    """A V row that is not finite reaches no query before it under the causal
    mask, within one key tile and across tiles."""
    n, H, hd = 70, 2, 32
    at = 41
    g = np.random.default_rng(5)
    t = to_dev(g.standard_normal((n, 3 * H * hd)).astype(np.float32), "f32")
    q, k, v = t.split(H * hd, dim=1)
    seqs = zsa.Seqs([n], dev())
    ref = zsa.attention_with_scores(q, k, v, H, seqs, True)[0].clone()
    v[at] = bad
    out = zsa.attention_with_scores(q, k, v, H, seqs, True)[0]
    assert_close(f64(out)[:at], f64(ref)[:at], 1e-6, "rows before the one that is not finite")
    assert not torch.isfinite(out[at:]).any()


@pytest.mark.parametrize("hd", [16, 64])
@pytest.mark.parametrize("top,first", [(0, 1), (0, 32), (140, 1)])  # special keys beside the top one, in another
def test_attention_f32_small_probabilities(hd, top, first):         # wave's tile, and before it in the same wave
    """Probabilities down to e^-48 keep fp32's relative precision. Query 0's
    scores are exact (one product each): 0 for key ``top``, -x for 16 special
    keys, -200 for the rest, so its sum rounds to 1 and its log-sum-exp to 0
    and every exponent is exact. Each special key has a V channel to itself
    and, as the other queries' scores are four times as low, a contribution
    score of e^-x (1 + 1e-14). Bounds, with u = 2^-24: an exponential is
    within 2u; at most three of them and three products make a probability;
    the sums add terms below 1e-9: 10 u = 6e-7. (An exponential that rounds
    its argument times log2 e to fp32 is off by up to 2^-24 times that
    argument, 58 here.)"""
    n, x = 150, 18.0 + 2.0 * np.arange(16) - 0.0625 * np.arange(16) ** 2 + np.linspace(0, 15, 16)
    x = np.float32(np.round(x * 64) / 64)
    qkv = np.zeros((n, 3 * hd), dtype=np.float32)
    qkv[:, 0] = 4.0
    qkv[0, 0] = 1.0
    qkv[:, hd] = -200.0
    qkv[top, hd] = 0.0
    qkv[first:first + 16, hd] = -x
    qkv[first + np.arange(16), 2 * hd + np.arange(16)] = 1.0
    q, k, v = to_dev(qkv, "f32").split(hd, dim=1)
    out, lse, scores = zsa.attention_with_scores(q, k, v, 1, zsa.Seqs([n], dev()), False, scale=1.0)
    p = np.exp(-x.astype(np.float64))
    assert abs(f64(lse)[0, 0]) <= 3e-7  # the sum of the others, and one rounding
    assert np.abs(f64(out)[0, :16] / p - 1.0).max() <= 6e-7
    assert np.abs(f64(scores)[first:first + 16] / p - 1.0).max() <= 6e-7
