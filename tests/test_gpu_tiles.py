"""GEMM tile shapes through the C ABI (GPU).

The GEMM tile is chosen from the row count, so one stream runs other kernels
than a batch.  Every tile shape of a type sums in the same order: a stream's
velocity must be bitwise the same at every batch size, and the single
stream's must match the oracle (half of the latent bar of the type, 2e-2 in
bf16 and 1e-4 in fp32, as in the other single-evaluation tests at larger
widths)."""
import dataclasses

import numpy as np
import pytest

from oracle import dit
from paper_2607_23159_amd import synth

from parity import TOL, rel_l2

pytestmark = pytest.mark.gpu


# tokens: one row short of and past tile edges, below one tile, and the
# ragged geometry; batches reach from 32 x 32 tiles to 256 x 256 ones
GRIDS = [
    ("tiny", (1, 3, 5), (1, 2, 5, 64)),            # 15 rows: less than any tile; K of one and two slices
    ("ragged", (3, 9, 11), (1, 3, 17, 90)),        # 297 rows
    ("wan_mid", (1, 5, 13), (1, 2, 31)),           # 65 rows: one past a 64-row tile; K = 8960 is 140 slices
    ("wan_mid", (3, 8, 16), (1, 4, 9, 33)),        # 384 rows to 12,672: 64 to 256-row tiles
]
# 391 rows, an odd number: 192, 224 and 256-row tiles whose waves store their rows
# and the transposed values through LDS (tests/test_gemm_tile_choice.py holds both
# lists to the library's tile choice)
STAGED_GRIDS = [
    ("wan_mid", (1, 17, 23), (1, 6, 7, 13)),
    ("wan5b_mid", (1, 17, 23), (1, 2, 3)),
    ("wan14b_mid", (1, 17, 23), (1, 2, 4)),
]


@pytest.mark.parametrize("dtype", [synth.DTYPE_BF16, synth.DTYPE_FP32])
@pytest.mark.parametrize("model,grid,batches", GRIDS)
def test_velocity_is_bitwise_the_same_at_every_batch_size(model, grid, batches, dtype):
    same_at_every_batch_size(model, grid, batches, dtype)


@pytest.mark.parametrize("model,grid,batches", STAGED_GRIDS)
def test_velocity_is_bitwise_the_same_with_large_tiles(model, grid, batches):
    same_at_every_batch_size(model, grid, batches, synth.DTYPE_BF16)


# fp32 attention at head dims 32 and 64: one stream takes one block of 32 queries
# per wave, the batch (512 and 432 workgroups of one block, two rounds of 256 CUs,
# against one of 64) two.  The last workgroup's second block holds one query (225,
# 289 tokens) or none (259).
@pytest.mark.parametrize("model,grid,batches", [
    ("tiny", (1, 15, 15), (1, 16)),
    ("tiny", (1, 7, 37), (1, 12)),
    ("ragged", (1, 17, 17), (1, 12)),
])
def test_velocity_with_two_query_blocks_per_wave(model, grid, batches):
    same_at_every_batch_size(model, grid, batches, synth.DTYPE_FP32)


def same_at_every_batch_size(model, grid, batches, dtype):
    import torch

    from paper_2607_23159_amd.search import GpuModel
    f, h, w = grid
    m = dataclasses.replace(synth.MODELS[model], n_blocks=1, lat_f=f, lat_h=2 * h, lat_w=2 * w,
                            dtype=dtype)
    weights = synth.make_weights(m, seed=5, init="stress", std=0.03)
    gm = GpuModel(m, weights)
    x = torch.from_numpy(synth.make_noise(m, max(batches), seed0=40)).cuda()
    ctx = synth.make_context(m, 9)
    ctx_d = torch.from_numpy(ctx).cuda()
    ref = gm.velocity(x[:1].contiguous(), 0.4, ctx_d)
    W = {k: v.astype(np.float64) for k, v in synth.unflatten(m, weights).items()}
    exp = dit.velocity(x[0].cpu().numpy(), np.float32(0.4), dit.text_embedding(ctx, W), W, m)
    assert rel_l2(ref[0].cpu().numpy(), exp) < TOL[dtype] / 2
    for n in batches[1:]:
        # the first stream repeated at both ends of the batch
        xb = x[:n].clone()
        xb[-1] = x[0]
        v = gm.velocity(xb, 0.4, ctx_d)
        assert torch.isfinite(v).all()
        assert torch.equal(v[0], ref[0]) and torch.equal(v[-1], ref[0]), f"batch of {n}"
    gm.close()
