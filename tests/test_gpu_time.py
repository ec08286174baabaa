"""Order of the time conditioning's sums through the C ABI (GPU).

The three matrix-vector products of the time conditioning sum in one fixed
order: 64 partial sums, sum c over the columns k = c mod 64 in increasing k
with fused multiply-adds, added in halves (c and c + 32, then 16, 8, 4, 2, 1),
then the bias.  A bf16 evaluation multiplies a last-bit change of a modulation
vector by 1e4, so the order is pinned bit for bit: the expected vectors are
formed in that order on the CPU, the modulation tables of the model are set to
minus them, and a model whose other weights are zero must then return exactly
zero (the head's shift and the blocks' gates vanish, and any other value
reaches the velocity).

At t = 0 the features are exactly 1 (cosines) and 0 (sines), and every hidden
value lies above 18, where SiLU returns its argument (1 + e^-18 rounds to 1).
"""
import dataclasses

import numpy as np
import pytest

from paper_2607_23159_amd import synth

pytestmark = pytest.mark.gpu


def gemv(w, x, b):
    """w x + b with the library's order; products and sums in 64 mantissa
    bits, rounded to fp32 after every step like a fused multiply-add."""
    n, k = w.shape
    w = w.astype(np.longdouble).reshape(n, k // 64, 64)
    x = x.astype(np.longdouble).reshape(k // 64, 64)
    s = np.zeros((n, 64), np.float32)
    for j in range(k // 64):
        s = (w[:, j] * x[j] + s).astype(np.float32)
    for o in (32, 16, 8, 4, 2, 1):
        s = s[:, :o] + s[:, o:]
    return s[:, 0] + b


@pytest.mark.parametrize("dtype", [synth.DTYPE_BF16, synth.DTYPE_FP32])
# widths: two and four steps of 64 columns, 24 (whole groups of eight), 5 (odd);
# more blocks than the eight lanes of a row
@pytest.mark.parametrize("model,heads,blocks", [("tiny", 4, 10), ("ragged", 4, 2), ("wan_mid", 12, 1),
                                                ("ragged", 5, 9)])
def test_time_conditioning_sums_in_one_fixed_order(model, heads, blocks, dtype):
    import torch

    from paper_2607_23159_amd.search import GpuModel
    base = synth.MODELS[model]
    m = dataclasses.replace(base, n_blocks=blocks, heads=heads, hidden=heads * base.head_dim, lat_f=1, lat_h=4,
                            lat_w=6, text_len=8, dtype=dtype)
    d, rng = m.hidden, np.random.default_rng(7)
    weights = np.zeros(synth.weight_count(m), np.float32)
    W = synth.unflatten(m, weights)

    def matrix(name, cols, total):
        # positive with a mean of total / cols: the sums grow to `total`, and
        # every step rounds; bf16 values, exact in both types
        v = (total / cols * (1 + 0.3 * rng.standard_normal(W[name].shape[:1] + (cols,)))).astype(np.float32)
        v = torch.from_numpy(v).bfloat16().float().numpy()
        W[name][:, :cols] = v

    half = m.freq_dim // 2
    matrix("time1_w", half, 40.0)
    W["time1_w"][:, half:] = rng.integers(-3, 4, (d, half))
    matrix("time2_w", d, 1.0)
    matrix("mod_w", d, 1.0)
    for name in ("time1_b", "time2_b", "mod_b"):
        W[name][:] = rng.standard_normal(W[name].shape).astype(np.float32)
    feat = np.concatenate([np.ones(half, np.float32), np.zeros(half, np.float32)])
    h = gemv(W["time1_w"], feat, W["time1_b"])
    e = gemv(W["time2_w"], h, W["time2_b"])
    mod = gemv(W["mod_w"], e, W["mod_b"])
    assert min(h.min(), e.min()) > 18
    for j in range(blocks):
        b = f"blk{j}."
        W[b + "mod"][:] = -mod.reshape(6, d)
        for name in ("q_gain", "k_gain", "ca_ln_g", "caq_gain", "cak_gain", "o_b", "ffn2_b"):
            W[b + name][:] = 1.0
    W["head_mod"][:] = -e
    W["head_w"][:] = rng.standard_normal(W["head_w"].shape)
    gm = GpuModel(m, weights)
    x = torch.from_numpy(synth.make_noise(m, 1)).cuda()
    ctx = torch.from_numpy(synth.make_context(m, 9)).cuda()
    v = gm.velocity(x, 0.0, ctx)
    gm.close()
    assert torch.count_nonzero(v) == 0, f"largest deviation {v.abs().max().item():.3e}"
