"""split_k = 1 with a tile id: a matrix's result is the same bits alone, among others
and in batches that pass the sizes at which a call's tiles, operand rings, norm
items, last rounds and the one-kernel path change."""
import numpy as np
import pytest

import synth
from tests.gpu_util import oracle_schedule

pytestmark = pytest.mark.gpu


def _same(shape, count, others=(), dtype="bfloat16", seed=1, **kw):
    import torch
    import paper_2505_16932_amd as pe
    dt = getattr(torch, dtype)
    mk = lambda sh, k: torch.from_numpy(synth.rng(seed + k).standard_normal(sh).astype(np.float32)).cuda().to(dt)
    G = mk(shape, 0)
    kw = dict(dict(T=4, abc=oracle_schedule(4), out_dtype=torch.float32, split_k=1), **kw)
    alone = pe.polar_batched([G], **kw)[0]
    many = pe.polar_batched([G] * count + [mk(sh, 1 + k) for k, sh in enumerate(others)], **kw)
    torch.cuda.synchronize()
    for k in (0, count // 2, count - 1):
        assert torch.equal(alone, many[k]), (shape, count, k, kw)


@pytest.mark.parametrize("compute", ["bf16", "f32"])
@pytest.mark.parametrize("shape,count,others", [
    ((512, 512), 20, ()),                       # 64 tiles alone, 128 tiles in a call of 320
    ((1024, 1024), 6, ()),                      # update on 64 or 128 tiles
    ((1000, 2000), 12, ()),                     # deep and shallow rings, symmetric tiles
    ((700, 1500), 1, [(60, 300), (2000, 2000), (9, 70)]),
    ((1600, 1700), 5, [(100, 3000)]),
    ((60, 900), 2, [(300, 300)]),               # the one-kernel path, beside a matrix that does not fit
    ((64, 500), 70, [(256, 256)]),
])
def test_small_tiles(shape, count, others, compute):
    _same(shape, count, others, compute=compute, tile=1, dtype="float32" if compute == "f32" else "bfloat16")


@pytest.mark.parametrize("shape,count,others", [
    ((512, 2048), 17, ()),                      # a short last round
    ((512, 2048), 20, [(700, 300)]),
    ((1500, 1100), 12, ()),
    ((300, 700), 50, ()),
])
def test_large_tile(shape, count, others):
    _same(shape, count, others, tile=2)


@pytest.mark.parametrize("shape,count", [((1024, 2048), 16), ((300, 900), 80), ((2000, 2100), 4)])
def test_fast_iteration(shape, count):
    _same(shape, count, dtype="float32", compute="f32", fast_restart=2, tile=1)


@pytest.mark.parametrize("compute,tile", [("bf16", 1), ("bf16", 2), ("f32", 1)])
def test_spectral_init(compute, tile):
    _same((700, 900), 40, [(1100, 300)], compute=compute, tile=tile, spectral_init=6,
          dtype="float32" if compute == "f32" else "bfloat16")


@pytest.mark.parametrize("shape", [(64, 64), (200, 900), (500, 250)])
def test_library_choice_of_small_matrices(shape):
    """(Up to s = 256 every regime gives the small tiles.)"""
    _same(shape, 60, [(400, 100)])
