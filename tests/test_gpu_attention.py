"""bf16 attention at the edges of the long-sequence kernel's tiles (32-key
steps, 64-key tiles, 256-query blocks) and of the order its workgroups are
placed in, against the float64 oracle. Two bf16 roundings reach the output,
that of each probability and its own, each at most u = 2^-8 relative: element
by element |error| <= u (sum_j p_j |v_j| + |o|), the first sum being the
attention of |v|, plus fp32 sums (1 %). The log-sum-exp is held to 1e-5 and the
scores to 1e-4 (fp32 sums), as in the other attention tests."""
import math

import numpy as np
import pytest
import torch

from oracle import zsa_oracle as O
from paper_2509_01190_amd import zsa
from tests.helpers import assert_close, dev, f64, score_err, to_dev

pytestmark = pytest.mark.gpu


def check(lens, H, hkv, hd, causal, seed, sharp=1.5, shape_scores=None):
    g = np.random.default_rng(seed)
    T, d, kvd = sum(lens), H * hd, hkv * hd
    a = g.standard_normal((T, d + 2 * kvd)).astype(np.float32)
    a[:, :d] *= sharp
    if shape_scores is not None:
        a = shape_scores(a, d, kvd)
    q, k, v = to_dev(a, "bf16").split([d, kvd, kvd], dim=1)
    seqs = zsa.Seqs(lens, dev())
    out, lse, scores = zsa.attention_with_scores(q, k, v, H, seqs, causal, n_kv_heads=hkv)
    q64, k64, v64 = (f64(t) for t in (q, k, v))
    k64, v64 = (np.repeat(t.reshape(T, hkv, hd), H // hkv, axis=1).reshape(T, d) for t in (k64, v64))
    for b, n in enumerate(lens):
        if n == 0:
            continue
        s = slice(int(seqs.host[b]), int(seqs.host[b + 1]))
        o, l, sc = O.attention(q64[s], k64[s], v64[s], np.arange(n), H, causal)
        av, _, _ = O.attention(q64[s], k64[s], np.abs(v64[s]), np.arange(n), H, causal)
        off = np.abs(f64(out)[s] - o) / (2.0 ** -8 * (av + np.abs(o)))
        assert off.max() <= 1.01, f"attention, {n} rows: {off.max():.3f} of the rounding bound"
        assert_close(f64(lse)[:, s], l, 1e-5, f"log-sum-exp, {n} rows")
        assert score_err(f64(scores)[s], sc) <= 1e-4


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("lens,H,hkv", [([385], 1, 1),                      # one pair: seven XCDs idle
                                        ([512, 512, 512], 8, 2),            # equal lengths, whole tiles
                                        ([575, 576, 577, 0, 1, 33, 64], 3, 1),  # tile edges, ragged, empty
                                        ([449, 449], 12, 12),               # heads not a multiple of 8
                                        ([801, 40, 769], 16, 4),            # two heads per XCD, shared keys
                                        ([(97 * i) % 331 for i in range(40)] + [600], 16, 4)])  # the scores' long grid
def test_attention_tiles_and_order(hd, causal, lens, H, hkv):
    check(lens, H, hkv, hd, causal, seed=hd + H + causal)


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("lens,H,hkv", [([575, 576, 577, 0, 1, 33, 64, 449], 12, 4),  # tile edges, ragged, empty
                                        ([512] * 5, 32, 32)])                         # whole tiles, heads in plain order
def test_attention_causal_full_grid(hd, lens, H, hkv):
    """Grids of more 256-query blocks than CUs, from where on head dim 64
    takes the long-sequence kernel under the mask (and 128 up to 512 rows)."""
    check(lens, H, hkv, hd, True, seed=hd + H)


@pytest.mark.parametrize("hd", [64, 128])
def test_attention_moving_reference_full_grid(hd):
    """As below, on such a grid."""
    def rise(a, d, kvd):
        i = np.arange(a.shape[0]) % 700
        a[:, d:d + kvd] *= 0.2
        a[:, d] = np.floor(i / 100.0) * 3.0
        a[:, 0] = np.where(i % 3 == 0, 8.0 * math.sqrt(hd) / 8.0, 0.1)
        return a
    check([700] * 6, 16, 16, hd, True, seed=13 + hd, sharp=1.0, shape_scores=rise)


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("causal", [False, True])
def test_attention_moving_reference(hd, causal):
    """Keys whose scores rise in steps along the sequence, far enough (20 exp2
    units and more) that the probabilities pass the bound and the reference
    moves in the middle, for some queries and not for others."""
    def rise(a, d, kvd):
        n = a.shape[0]
        a[:, d:d + kvd] *= 0.2
        a[:, d] = np.floor(np.arange(n) / 100.0) * 3.0   # channel 0 of head 0
        a[:, 0] = np.where(np.arange(n) % 3 == 0, 8.0 * math.sqrt(hd) / 8.0, 0.1)
        return a
    check([700], 2, 2, hd, causal, seed=11 + hd, sharp=1.0, shape_scores=rise)


def test_attention_many_equal_sequences():
    """More equal sequences of two rows, unmasked, than a grid's z holds at one
    chunk of heads each (12 heads: 43,690): the bounds of check()."""
    n, H, hd = 44000, 12, 64
    g = torch.Generator(device=dev()).manual_seed(3)
    q, k, v = torch.randn((2 * n, 3 * H * hd), generator=g, device=dev()).to(torch.bfloat16).split(H * hd, dim=1)
    out, lse, scores = zsa.attention_with_scores(q, k, v, H, zsa.Seqs([2] * n, dev()), False)
    q64, k64, v64 = (t.to(torch.float64).reshape(n, 2, H, hd) for t in (q, k, v))
    s = torch.stack([(q64 * k64[:, j:j + 1]).sum(dim=3) for j in (0, 1)], dim=3) / math.sqrt(hd)  # [n, 2, H, key]
    l = torch.logsumexp(s, dim=3)
    p = torch.exp(s - l[..., None])
    o = sum(p[..., j:j + 1] * v64[:, j:j + 1] for j in (0, 1))
    av = sum(p[..., j:j + 1] * v64[:, j:j + 1].abs() for j in (0, 1))
    off = (out.to(torch.float64).reshape(n, 2, H, hd) - o).abs() / (2.0 ** -8 * (av + o.abs()))
    assert off.max().item() <= 1.01
    l = l.reshape(2 * n, H).t()
    assert ((lse.to(torch.float64) - l).abs() / l.abs().clamp(min=1.0)).max().item() <= 1e-5
    sc = p.sum(dim=(1, 2)).reshape(-1)
    assert ((scores.to(torch.float64) - sc).abs() / sc.clamp(min=1.0)).max().item() <= 1e-4
