"""The LM head's position tiles: launches of different sizes take tiles of 64,
128 or 256 positions (fp32: 16, 32 or 64), and a row's statistics must
not depend on which."""
import numpy as np
import pytest
import torch

import oracle
from paper_2609_39859_amd import _binding
from harness import Report, compare_sampled, compare_stats, gpu_step, host_bits, record

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0")


def _inputs(M, d, V, seed, dtype=torch.bfloat16):
    g = torch.Generator().manual_seed(seed)
    W = (torch.randn(V, d, generator=g) / d ** 0.5).to(dtype)
    h = (torch.randn(M, d, generator=g) * (0.5 + 1.5 * torch.rand(M, 1, generator=g))).to(dtype)
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


# fp32: edges of the 16-position columns, of a wave's 32 rows, of the tile, of
# the K stages (32 elements) and of the 16-byte chunks
@pytest.mark.parametrize("M", [1, 16, 17, 130])
@pytest.mark.parametrize("d,V", [(4, 1), (32, 31), (36, 33), (132, 255), (256, 257), (68, 600)])
def test_f32_tile_edges_match_oracle(M, d, V):
    h, W = _inputs(M, d, V, M * 1000 + V, torch.float32)
    g = _step(h, W)
    ref = oracle.row_stats(host_bits(h), host_bits(W))
    rep = Report()
    compare_stats(g, ref, np.arange(M), host_bits(h), host_bits(W), d, rep)
    record(rep, "tiles_f32")


# a ragged vocabulary tile: its last block, half and row, one row in all
@pytest.mark.parametrize("V", [1, 15, 17, 127, 128, 130, 255, 300])
@pytest.mark.parametrize("M,dtype", [(70, torch.bfloat16), (700, torch.bfloat16),
                                     (70, torch.float32)])
def test_drawn_candidates_of_a_ragged_tile(V, M, dtype):
    d, rows = 72, np.arange(70)
    h, W = _inputs(M, d, V, M + V, dtype)
    g = _step(h, W, 0.8)
    hb, Wb = host_bits(h), host_bits(W)
    st = oracle.row_stats(hb, Wb, rows)
    sm = oracle.row_sample(hb, Wb, rows, 0.8, 11, 2)
    rep = Report()
    compare_sampled(g, st, sm, rows, hb, Wb, d, 0.8, 11, 2, rep)
    record(rep, "tiles_drawn")


# V = 32000 (125 vocabulary tiles): 1024 rows take tiles of 256 positions, 160
# rows tiles of 128, 40 rows tiles of 64; V = 2000 takes 64 throughout; V = 70000
# (274): 40 and 64 rows tiles of 64 two to a CU, on its shorter W ring; fp32
# tiles of 16, 32, 64 alone on a CU and 64 two to a CU, then (274 vocabulary
# tiles) 16, 32 and 64 two to a CU
@pytest.mark.parametrize("V,sizes,dtype", [(32000, (40, 160, 1024), torch.bfloat16),
                                           (2000, (3, 70, 300), torch.bfloat16),
                                           (70000, (40, 64, 1024), torch.bfloat16),
                                           (32000, (16, 48, 128, 256), torch.float32),
                                           (70000, (16, 32, 300), torch.float32)])
@pytest.mark.parametrize("temperature", [0.0, 0.8])
@pytest.mark.parametrize("d", [32, 72, 264])  # one stage (fp32: three tiles to a CU), and more
def test_rows_do_not_depend_on_the_tile(V, sizes, dtype, temperature, d):
    h, W = _inputs(max(sizes), d, V, V, dtype)
    outs = [_step(h[:n].contiguous(), W, temperature) for n in sizes]
    for n, g in zip(sizes[:-1], outs[:-1]):
        for k in ("conf", "entropy", "logp", "lse", "argmax"):
            a, b = getattr(g, k), getattr(outs[-1], k)[:n]
            assert np.array_equal(a.view(np.int32), b.view(np.int32)), (k, n)


# 788, 260 and 288 tiles of 256 positions: the 20, 4 and 32 past the whole
# rounds of 256 run as quarters, the last positions and words among them
@pytest.mark.parametrize("M,d,V", [(903, 72, 50257), (1030, 40, 13300), (2100, 64, 8000)])
def test_quartered_tail_matches_whole_tiles(M, d, V):
    h, W = _inputs(M, d, V, M)
    full = {t: _step(h, W, t) for t in (0.0, 0.8)}
    for rows, temperature in ((slice(0, 700), 0.0), (slice(0, 700), 0.8),
                              (slice(M - 60, M), 0.0)):  # draws depend on the row's index
        g = _step(h[rows].contiguous(), W, temperature)
        for k in ("conf", "entropy", "logp", "lse", "argmax"):
            a, b = getattr(g, k), getattr(full[temperature], k)[rows]
            assert np.array_equal(a.view(np.int32), b.view(np.int32)), (k, rows, temperature)
    hd, Wd = h.to(DEV), W.to(DEV)
    toks = torch.arange(M, dtype=torch.int32, device=DEV) * 7919 % V
    lp = torch.zeros(M, device=DEV)
    _binding.logprob(hd, Wd, toks, lp)
    for rows in (slice(0, 700), slice(M - 60, M)):
        part = torch.zeros_like(lp[rows])
        _binding.logprob(hd[rows].contiguous(), Wd, toks[rows].contiguous(), part)
        assert torch.equal(part.view(torch.int32), lp[rows].view(torch.int32)), rows


@pytest.mark.parametrize("B,BL,d,V", [(206, 5, 40, 13300), (43, 21, 72, 50257)])
def test_quartered_tail_through_a_row_list(B, BL, d, V):
    """The same tiles with the positions gathered: the active blocks, greedy and
    drawn, and given rows' likelihoods, against the same rows without a list."""
    L, tau = 2 * BL, 0.9
    h, W = _inputs(B * L, d, V, B)
    hd, Wd = h.to(DEV), W.to(DEV)
    rng = np.random.default_rng(B)
    bs = rng.integers(0, 2, B) * BL
    mask = np.ones(B * L, np.uint8)
    mask.reshape(B, L)[5] = 0                              # no rows of this sequence
    rows = (np.arange(B)[:, None] * L + bs[:, None] + np.arange(BL))[np.arange(B) != 5].ravel()
    for temperature in (0.0, 0.8):
        out = [gpu_step(hd, Wd, np.full(B * L, -1), mask, bs, B, L, BL, tau, rows_mode=mode,
                        temperature=temperature, seed=11, counter=2)
               for mode in (_binding.FORK_ROWS_ACTIVE, _binding.FORK_ROWS_ALL)]
        for k in ("conf", "entropy", "logp", "lse", "argmax"):
            a, b = (getattr(g, k)[rows] for g in out)
            assert np.array_equal(a.view(np.int32), b.view(np.int32)), (k, temperature)
    pick = torch.as_tensor(rng.permutation(B * L)[:B * BL].astype(np.int32)).to(DEV)
    toks = torch.as_tensor(rng.integers(0, V, B * BL).astype(np.int32)).to(DEV)
    a, b = torch.zeros(B * BL, device=DEV), torch.zeros(B * BL, device=DEV)
    _binding.logprob(hd, Wd, toks, a, rows=pick)
    _binding.logprob(hd[pick.long()].contiguous(), Wd, toks, b)
    assert torch.equal(a.view(torch.int32), b.view(torch.int32))
