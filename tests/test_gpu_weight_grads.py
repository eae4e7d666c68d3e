"""Weight, bias, gain and shift gradients where their kernels' shapes end: the
product dY^T X at the edges of its 64-, 128- and 256-wide tiles, one row, rows that
are no multiple of a slice, several row splits, and column counts below a
tile; the norm's column sums with one row and with more rows than workgroups;
the compaction's scatter with rows kept at either end."""
import numpy as np
import pytest
import torch

from oracle import zsa_grad as G
from paper_2509_01190_amd import workloads as W
from paper_2509_01190_amd import zsa
from tests.helpers import dev, f64, rel_l2, to_dev, weights_f64
from tests.test_gpu_stack import build, gpu_kept_overrides

pytestmark = pytest.mark.gpu

CASES = [
    # kind, heads, head_dim, d_ff, lengths, pruned
    (W.ENCODER, 1, 64, 72, [1], False),               # one row, d_ff just past a tile
    (W.DECODER, 3, 64, 40, [65, 7], True),            # 192 columns, d_ff below a tile
    (W.ENCODER, 1, 128, 136, [700, 323], True),       # several row splits, a short last one
    (W.DECODER, 8, 128, 520, [131], False),           # 128-wide tiles: 3072 x 1024, 1040 x 1024
    (W.ENCODER, 9, 64, 2056, [300, 1, 90], True),     # 128-wide tiles with a remainder both ways
    (W.DECODER, 9, 128, 6560, [130, 33], True),       # 256-wide tiles, remainders
    (W.ENCODER, 33, 128, 136, [40, 5], True),         # rows shared by four waves, the widest
    (W.DECODER, 17, 128, 72, [9], False),             # ... and the narrowest
]


@pytest.mark.parametrize("kind,heads,hd,ff,lens,prune", CASES)
def test_weight_gradients(kind, heads, hd, ff, lens, prune):
    p = W.shrink(W.PRESETS["dec1b"], kind=kind, causal=kind == W.DECODER, n_layers=1,
                 d_model=heads * hd, n_heads=heads, d_ff=ff, batch=len(lens),
                 prune_after=(1,) if prune else (), n_kv_heads=0)
    lens, stack, xd, posd, dws, ocfg = build(p, 5, lens, sharp=2.0)
    seqs = zsa.Seqs(lens, dev())
    rates = [0.4] * len(lens)
    out = stack.forward(xd, posd, seqs, p.prune_after, rates, debug=True)
    g = np.random.default_rng(3)
    dy = to_dev(g.standard_normal((out["t_final"], p.d_model)).astype(np.float32), "bf16")
    dx, grads = stack.backward(xd, posd, seqs, p.prune_after, rates, dy)
    torch.cuda.synchronize()
    over = gpu_kept_overrides(p, lens, seqs, out) if prune else [{} for _ in lens]
    x_all, dy_all, ws64 = f64(xd), f64(dy), [weights_f64(w) for w in dws]
    ref, ref_dx = None, []
    for b, n in enumerate(lens):
        lo, fo, fe = int(seqs.host[b]), out["cu_host"][b], out["cu_host"][b + 1]
        kept = {l: v[0] for l, v in over[b].items()}
        _, rdx, rg = G.stack_backward(x_all[lo:lo + n], np.arange(n), ws64, ocfg, p.prune_after,
                                      kept, dy_all[fo:fe])
        ref_dx.append(rdx)
        ref = rg[0] if ref is None else {k: None if v is None else ref[k] + v for k, v in rg[0].items()}
    # bf16 activations and gradients between the kernels, one layer: a few
    # roundings of 2^-9 each (the three-layer test's bound)
    assert rel_l2(f64(dx), np.concatenate(ref_dx)) <= 2e-2
    for name, v in ref.items():
        if v is None or grads[0][name] is None:
            continue
        got = grads[0][name].cpu().double().numpy()
        if np.linalg.norm(v) == 0:
            assert np.linalg.norm(got) == 0, name
        elif sum(lens) == 1 and name == "w_qkv":
            # one row: the softmax is 1, so the query and key gradients vanish
            lim = p.d_model * 2
            assert rel_l2(got[lim:], v[lim:]) <= 2e-2
        elif sum(lens) == 1 and name == "b_qkv":
            assert rel_l2(got[p.d_model * 2:], v[p.d_model * 2:]) <= 2e-2
        else:
            assert rel_l2(got, v) <= 2e-2, name


@pytest.mark.parametrize("d,ff,rows", [(768, 3072, 4000),   # 128-wide tiles, three row splits
                                       (768, 768, 4000),    # 64-wide
                                       (2048, 8192, 2100)]) # 256-wide
def test_bias_gradient_precision(d, ff, rows):
    """The down projection's bias gradient is the column sums of dy, whose
    bf16 rows are given: of the same sign, where the roundings of a long chain
    of additions add up. In levels the sums stay within one unit, 2^-24, of
    the 64-bit ones (2-norm over the columns); in one chain per wave they were
    8.0e-8 off at the first size."""
    p = W.shrink(W.PRESETS["dec1b"], kind=W.ENCODER, causal=False, n_layers=1, d_model=d, n_heads=d // 64,
                 d_ff=ff, batch=rows // 100, prune_after=(), n_kv_heads=0)
    lens, stack, xd, posd, _, _ = build(p, 5, [100] * (rows // 100), sharp=2.0)
    g = np.random.default_rng(7)
    dy = to_dev(np.abs(g.standard_normal((sum(lens), d))).astype(np.float32), "bf16")
    _, grads = stack.backward(xd, posd, zsa.Seqs(lens, dev()), (), [1.0] * len(lens), dy)
    assert rel_l2(f64(grads[0]["b_down"]), f64(dy).sum(axis=0)) <= 2.0 ** -24
