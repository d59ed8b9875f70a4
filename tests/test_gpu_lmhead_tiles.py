"""The LM head's position tiles: launches of different sizes take tiles of 64,
128 or 256 positions, and a row's statistics must not depend on which."""
import numpy as np
import pytest
import torch

import oracle
from harness import Report, compare_stats, gpu_step, host_bits, record

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0")


def _inputs(M, d, V, seed):
    g = torch.Generator().manual_seed(seed)
    W = (torch.randn(V, d, generator=g) / d ** 0.5).bfloat16()
    h = (torch.randn(M, d, generator=g) * (0.5 + 1.5 * torch.rand(M, 1, generator=g))).bfloat16()
    return h, W


def _step(h, W, temperature=0.0):
    """All rows of one sequence, every position masked."""
    M = h.shape[0]
    return gpu_step(h.to(DEV), W.to(DEV), np.full(M, -1), np.ones(M, np.uint8), np.zeros(1),
                    1, M, M, 0.9, temperature=temperature, seed=11, counter=2)


# edges of the position tiles (64, 128), of the vocabulary tile and its halves
# (128, 256), of the K stages (64 elements) and of the 16-byte chunks
@pytest.mark.parametrize("M", [1, 63, 64, 65, 129])
@pytest.mark.parametrize("d,V", [(8, 1), (64, 127), (72, 128), (136, 129), (1000, 255),
                                 (200, 256), (264, 257), (520, 641)])
def test_tile_edges_match_oracle(M, d, V):
    h, W = _inputs(M, d, V, M * 1000 + V)
    g = _step(h, W)
    ref = oracle.row_stats(host_bits(h), host_bits(W))
    rep = Report()
    compare_stats(g, ref, np.arange(M), host_bits(h), host_bits(W), d, rep)
    record(rep, "tiles")


# V = 32000 (125 vocabulary tiles): 1024 rows take tiles of 256 positions, 160
# rows tiles of 128, 40 rows tiles of 64; V = 2000 takes 64 throughout
@pytest.mark.parametrize("V,sizes", [(32000, (40, 160, 1024)), (2000, (3, 70, 300))])
@pytest.mark.parametrize("temperature", [0.0, 0.8])
def test_rows_do_not_depend_on_the_tile(V, sizes, temperature):
    d = 72
    h, W = _inputs(max(sizes), d, V, V)
    outs = [_step(h[:n].contiguous(), W, temperature) for n in sizes]
    for n, g in zip(sizes[:-1], outs[:-1]):
        for k in ("conf", "entropy", "logp", "lse", "argmax"):
            a, b = getattr(g, k), getattr(outs[-1], k)[:n]
            assert np.array_equal(a.view(np.int32), b.view(np.int32)), (k, n)
