"""Edges of the decode kernels that take all levels of a request in one workgroup, against the oracle."""
import numpy as np
import pytest
import torch

import synth
import paper_2511_18793_amd as nz
from _gpu_common import check_decode, planted_workload, to_device, tolerance

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,d,e,V,K,L,dtype", [
    (5, 64, 128, 528, 16, 3, "bf16"),     # one row tile, the first codebook past the small kernel's
    (3, 64, 32, 16, 16, 4, "bf16"),       # one column tile for eight waves
    (4, 64, 64, 144, 33, 3, "bf16"),      # a third row tile with one beam
    (3, 96, 96, 1040, 48, 3, "bf16"),     # three full row tiles, 65 column tiles
    (2, 64, 160, 256, 49, 2, "bf16"),     # a state between two instance widths
    (2, 64, 256, 320, 128, 3, "bf16"),    # eight row tiles, operands read from LDS
    (300, 32, 32, 544, 4, 3, "bf16"),     # more requests than compute units
    (7, 33, 32, 80, 9, 3, "f32"),
    (17, 65, 128, 256, 16, 3, "f32"),     # rows of A past the last full tile
    (2, 20, 256, 48, 33, 2, "f32"),
    (3, 64, 96, 512, 40, 2, "f32"),       # logits of a level past the LDS: the chunked kernel
])
@pytest.mark.parametrize("density", ["planted", "sparse"])
def test_decode_edges(oracle, B, d, e, V, K, L, dtype, density):
    cfg = synth.StepConfig("edge", B=B, d=d, e=e, L=L, V=V, K=K, N=min(V ** L // 4, 60_000), dtype=dtype,
                           catalog="uniform", w_std=0.05)
    x, cat = planted_workload(oracle, cfg, 5, plant=density == "planted")
    oset = oracle.ItemSet(cat, cfg.radices)
    H, W, E = to_device(x, cfg)
    outs = nz.decode(H, W, E, cfg.radices, cfg.K, nz.build_itemset(cat, cfg.radices))
    torch.cuda.synchronize()
    check_decode(oracle, nz, cfg, x, outs, oset, tolerance(cfg))


@pytest.mark.parametrize("n", [1, 255, 257, 70_001])
def test_build_counts_distinct_items(n):
    rng = np.random.default_rng(n)
    codes = rng.integers(0, 64, size=(n, 3), dtype=np.int32)
    gset = nz.build_itemset(np.concatenate([codes, codes[: n // 2]]), (64, 64, 64))
    assert gset.info()["n_distinct"] == len(np.unique(codes, axis=0))
