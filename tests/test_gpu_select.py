"""GPU parity of the unmasking rule on its own (fork_select, Algorithm 2 and
the fallback rules of Algorithm 1 and Section 4.1): its kernels (one wave per
sequence, one to eight lanes per sequence for large batches of short blocks,
and the position-major ones) against the oracle, bit for bit (both sides decide
on the same binary32 confidences)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2609_39859_amd import _binding

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0")


def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _state(B, L, V, seed):
    rng = np.random.default_rng(seed)
    M = B * L
    conf = rng.random(M).astype(np.float32)
    conf[rng.random(M) < 0.1] = np.float32(0.9)           # values on the threshold
    ent = np.round(rng.random(M) * 4, 2).astype(np.float32)  # frequent ties
    am = rng.integers(0, V, M).astype(np.int32)
    msk = (rng.random(M) < 0.5).astype(np.uint8)
    tok = np.where(msk, -1, rng.integers(0, V, M)).astype(np.int32)
    bs = rng.integers(0, L + 1, B).astype(np.int32)
    msk[(B - 1) * L:] = 0                                  # an idle sequence
    uni = rng.random(B).astype(np.float32)
    return conf, ent, am, tok, msk, bs, uni


def _pm(x, B, L):
    """Row-major [B*L] -> position-major [L*B] (position k of sequence b at
    k*B + b)."""
    return np.ascontiguousarray(np.asarray(x).reshape(B, L).T).reshape(-1)


def _rm(x, B, L):
    return np.ascontiguousarray(np.asarray(x).reshape(L, B).T).reshape(-1)


def _run(conf, ent, am, tok, msk, bs, uni, B, L, BL, tau, rule,
         layout=_binding.FORK_LAYOUT_ROW_MAJOR, outputs="all"):
    """fork_select on row-major host state; with the position-major layout
    the per-position arrays are transposed for the call and back after it,
    so the results compare directly.  outputs: "all" asks for the commit
    counts and positions, "ncommit" for the counts only, "none" for
    neither (their slots then come back as -9)."""
    t = lambda x: torch.as_tensor(np.ascontiguousarray(x), device=DEV)
    pm = layout == _binding.FORK_LAYOUT_POSITION_MAJOR
    lay = (lambda x: _pm(x, B, L)) if pm else (lambda x: x)
    tok_d, msk_d, bs_d = t(lay(tok).copy()), t(lay(msk).copy()), t(bs.copy())
    fb = torch.full((B,), -9, dtype=torch.int32, device=DEV)
    nc = torch.full((B,), -9, dtype=torch.int32, device=DEV)
    cp = torch.full((B * BL,), -9, dtype=torch.int32, device=DEV)
    _binding.select(t(lay(conf)), t(lay(am)), tok_d, msk_d, bs_d, BL, tau, fb, B=B, L=L,
                    rule=rule, entropy=t(lay(ent)), uniform=t(uni),
                    out_ncommit=nc if outputs in ("all", "ncommit") else None,
                    out_commit_pos=cp if outputs == "all" else None, layout=layout)
    torch.cuda.synchronize()
    back = (lambda x: _rm(x, B, L)) if pm else (lambda x: x)
    return (back(tok_d.cpu().numpy()), back(msk_d.cpu().numpy()), bs_d.cpu().numpy(),
            fb.cpu().numpy(), nc.cpu().numpy(), cp.cpu().numpy().reshape(B, BL))


SHAPES = [
    # B, L, block_len   (B >= 4096 with block_len <= 64: a group of lanes each)
    (5, 61, 7), (37, 300, 300), (4096, 40, 8), (5000, 64, 64), (4100, 33, 32),
    (4096, 100, 65), (4097, 1, 1),
    # lane groups with 16-byte aligned rows (wide loads)
    (4096, 32, 32), (4096, 64, 16), (8192, 96, 32), (4096, 48, 8),
]


PM_SHAPES = [
    # position-major: B % 4 == 0 with shared block starts takes the wide path
    (5, 61, 7), (6, 33, 32), (4096, 32, 32), (4096, 64, 16), (4100, 40, 8), (4099, 33, 32),
    (8, 100, 65), (4097, 1, 1), (1024, 48, 33),
]


@pytest.mark.parametrize("B,L,BL", SHAPES)
@pytest.mark.parametrize("rule", [0, 1, 2, 3, 4])
def test_select_matches_oracle(B, L, BL, rule):
    _check_against_oracle(B, L, BL, rule, _binding.FORK_LAYOUT_ROW_MAJOR)


@pytest.mark.parametrize("B,L,BL", PM_SHAPES)
@pytest.mark.parametrize("rule", [0, 1, 2, 3, 4])
@pytest.mark.parametrize("shared_start", [False, True])
def test_select_position_major_matches_oracle(B, L, BL, rule, shared_start):
    """The position-major layout against the oracle (on the transposed
    state), with random block starts and with every sequence at the same
    block start (the wide path)."""
    _check_against_oracle(B, L, BL, rule, _binding.FORK_LAYOUT_POSITION_MAJOR, shared_start)


def _check_against_oracle(B, L, BL, rule, layout, shared_start=False):
    _need_gpu()
    conf, ent, am, tok, msk, bs, uni = _state(B, L, 1000, B * 31 + L + BL + rule)
    if shared_start:
        bs[:] = min(L - BL, 3)
    for tau in (0.3, 0.9):
        g = _run(conf, ent, am, tok, msk, bs, uni, B, L, BL, tau, rule, layout)
        o = oracle.select_ex(conf, am, tok, msk, bs, B, L, BL, float(np.float32(tau)), rule,
                             entropy=ent, uniform=uni)
        for k, (x, y) in enumerate(zip(g[:5], o)):
            assert np.array_equal(x, y), ("tokens", "mask", "block_start", "fallback", "ncommit")[k]
        # compacted commits: the positions the oracle unmasked, ascending
        for b in range(B):
            sl = slice(b * L, (b + 1) * L)
            done = np.nonzero(msk[sl] & ~o[1][sl])[0]
            assert np.array_equal(g[5][b, :done.size], done)
            assert np.all(g[5][b, done.size:] == -1)


@pytest.mark.parametrize("B,L,BL", [(4096, 32, 32), (4096, 64, 16), (8192, 48, 8),
                                    (4160, 64, 32)])
@pytest.mark.parametrize("rule", [0, 4, 1])
@pytest.mark.parametrize("outputs", ["all", "none"])
def test_row_major_whole_wave_blocks(B, L, BL, rule, outputs):
    """Row-major batches whose blocks start on multiples of 16 positions
    with 32 positions left in the row (wide loads), one sequence in 128 off that
    grid (loads of single positions) and the last sequence idle, under the threshold, leftmost, random
    and highest-confidence rules, with and without the commit outputs.
    Against the oracle, bit for bit."""
    _need_gpu()
    conf, ent, am, tok, msk, bs, uni = _state(B, L, 1000, B + 7 * L + BL + rule)
    rng = np.random.default_rng(B + L + BL)
    bs[:] = rng.choice(np.arange(0, L - 32 + 1, 16), B)
    for w in range(1, B // 64, 2):
        bs[64 * w + 5] = min(bs[64 * w + 5] + 1, L)
    for tau in (0.3, 0.9):
        g = _run(conf, ent, am, tok, msk, bs, uni, B, L, BL, tau, rule, outputs=outputs)
        o = oracle.select_ex(conf, am, tok, msk, bs, B, L, BL, float(np.float32(tau)), rule,
                             entropy=ent, uniform=uni)
        n = 5 if outputs == "all" else 4
        for k, (x, y) in enumerate(zip(g[:n], o[:n])):
            assert np.array_equal(x, y), ("tokens", "mask", "block_start", "fallback", "ncommit")[k]
        if outputs == "all":
            for b in range(0, B, 97):
                sl = slice(b * L, (b + 1) * L)
                done = np.nonzero(msk[sl] & ~o[1][sl])[0]
                assert np.array_equal(g[5][b, :done.size], done)
                assert np.all(g[5][b, done.size:] == -1)


@pytest.mark.parametrize("L,BL", [(32, 32), (33, 31), (64, 32), (67, 33), (72, 40), (64, 64),
                                  (131, 63), (200, 64), (9, 5), (1, 1), (5, 2), (4, 4), (8, 8),
                                  (32, 8), (27, 7), (16, 16), (50, 9), (64, 16), (33, 17)])
@pytest.mark.parametrize("rule", [0, 1, 2, 3, 4])
def test_lane_groups_match_oracle(L, BL, rule):
    """Blocks around the lengths at which the lanes per sequence change (4, 8,
    16, 32), rows and starts on and off the 16-byte grid, blocks cut by the
    row's end, and a last workgroup that is not full."""
    _check_against_oracle(4099, L, BL, rule, _binding.FORK_LAYOUT_ROW_MAJOR)


@pytest.mark.parametrize("B,L,BL", [(16389, 32, 32), (16389, 32, 20), (16389, 64, 32), (16389, 99, 31),
                                    ((1 << 18) + 1, 33, 32), ((1 << 18) + 1, 21, 18),
                                    ((1 << 20) + 3, 32, 32)])
@pytest.mark.parametrize("rule", [0, 1, 2, 3, 4])
def test_large_batches_match_oracle(B, L, BL, rule):
    """Workgroups of 256, 128 and 64 sequences, and eight lanes per sequence on
    and off the 16-byte grid."""
    _need_gpu()
    _check_whole(_state(B, L, 1000, B + L + BL + rule), B, L, BL, rule, 0.9)


def test_more_sequences_than_a_launch_of_eight_lanes_each_holds():
    """2^29 sequences of one position: with eight lanes each a launch of 2^32
    work-items, which is refused."""
    _need_gpu()
    B = (1 << 29) + 5
    if torch.cuda.mem_get_info(DEV)[0] < 16 << 30:
        pytest.skip("needs 16 GB")
    i32 = dict(dtype=torch.int32, device=DEV)
    conf = torch.zeros(B, device=DEV)
    cand = torch.arange(B, **i32)
    tok, start, fb = torch.full((B,), -1, **i32), torch.zeros(B, **i32), torch.full((B,), -9, **i32)
    msk = torch.ones(B, dtype=torch.uint8, device=DEV)
    msk[::3] = 0
    _binding.select(conf, cand, tok, msk, start, 1, 0.5, fb, B=B, L=1, rule=1)
    torch.cuda.synchronize()
    assert not msk.any()
    assert bool((fb[::3] == -1).all()) and bool((fb[1::3] == 1).all()) and bool((fb[2::3] == 1).all())
    assert bool((tok[::3] == -1).all())
    assert torch.equal(tok[1::3], cand[1::3]) and torch.equal(tok[2::3], cand[2::3])


def _check_whole(state, B, L, BL, rule, tau, layout=_binding.FORK_LAYOUT_ROW_MAJOR):
    """Every output against the oracle, the committed positions of all
    sequences at once."""
    conf, ent, am, tok, msk, bs, uni = state
    g = _run(conf, ent, am, tok, msk, bs, uni, B, L, BL, tau, rule, layout)
    o = oracle.select_ex(conf, am, tok, msk, bs, B, L, BL, float(np.float32(tau)), rule,
                         entropy=ent, uniform=uni)
    for k, (x, y) in enumerate(zip(g[:5], o)):
        assert np.array_equal(x, y), ("tokens", "mask", "block_start", "fallback", "ncommit")[k]
    done = (msk != o[1]).reshape(B, L)
    want = np.full((B, BL), -1, np.int32)
    seq, where = np.nonzero(done)
    want[seq, (np.cumsum(done, axis=1) - 1)[seq, where]] = where
    assert np.array_equal(g[5], want)


def _nan_state(B, L, BL, rule):
    """Keys without a value above the threshold: NaN at the first masked
    position of the block, at random positions, and at all of them."""
    conf, ent, am, tok, msk, bs, uni = _state(B, L, 1000, B + 13 * L + BL + rule)
    conf = np.round(conf * 0.5, 2)                          # frequent ties
    rng = np.random.default_rng(B + L)
    bs[: B // 2] = rng.integers(0, L - BL + 1, B // 2)      # half the blocks whole
    key = (ent if rule == 3 else conf).reshape(B, L)
    m = msk.reshape(B, L)
    for b in range(min(B, 4200)):
        at = bs[b] + np.nonzero(m[b, bs[b]:])[0]
        if b % 3 == 0:
            key[b, at[:1]] = np.nan
        elif b % 3 == 1:
            key[b, rng.random(L) < 0.3] = np.nan
        else:
            key[b] = np.nan
    return conf, ent, am, tok, msk, bs, uni


@pytest.mark.parametrize("B,L,BL", [(4099, 32, 32), (4099, 67, 31), (4099, 64, 64), (4099, 131, 40),
                                    ((1 << 18) + 3, 32, 32), ((1 << 18) + 3, 37, 20), (4099, 4, 4),
                                    (4099, 7, 3), (4099, 16, 8), (4099, 40, 16), (4099, 45, 13)])
@pytest.mark.parametrize("rule", [1, 2, 3])
def test_nan_keys_follow_the_scan_in_order(B, L, BL, rule):
    """One to eight lanes per sequence, blocks up to 4, 8, 16, 32 and 64
    positions: one position is committed, the one a scan in order picks."""
    _need_gpu()
    _check_whole(_nan_state(B, L, BL, rule), B, L, BL, rule, 0.9)


@pytest.mark.parametrize("B,L,BL", [(60, 64, 64), (60, 67, 31), (60, 65, 65), (60, 400, 150)])
@pytest.mark.parametrize("layout", [_binding.FORK_LAYOUT_ROW_MAJOR,
                                    _binding.FORK_LAYOUT_POSITION_MAJOR])
@pytest.mark.parametrize("rule", [1, 2, 3])
def test_nan_keys_in_small_batches(B, L, BL, layout, rule):
    """One wave per sequence, blocks up to 64 positions and longer, and the
    position-major kernel."""
    _need_gpu()
    _check_whole(_nan_state(B, L, BL, rule), B, L, BL, rule, 0.9, layout)


def test_lane_and_wave_paths_agree():
    """The first sequences of a large batch (a group of lanes each) and the same
    sequences run as a small batch (a wave each) give identical results."""
    _need_gpu()
    B, L, BL = 4096, 64, 32
    conf, ent, am, tok, msk, bs, uni = _state(B, L, 500, 7)
    for rule in range(5):
        big = _run(conf, ent, am, tok, msk, bs, uni, B, L, BL, 0.5, rule)
        n = 64
        small = _run(conf[:n * L], ent[:n * L], am[:n * L], tok[:n * L], msk[:n * L], bs[:n],
                     uni[:n], n, L, BL, 0.5, rule)
        for x, y in zip(big, small):
            assert np.array_equal(x.reshape(-1)[:y.size], y.reshape(-1))


@pytest.mark.parametrize("B", [3, 4096])
def test_bad_block_start_reported_in_data_on_both_paths(B):
    _need_gpu()
    L, BL = 16, 4
    conf, ent, am, tok, msk, bs, uni = _state(B, L, 100, 3)
    msk[:] = 1
    bs[:] = 0
    bs[0], bs[1] = -1, L + 1
    bs[2] = L                           # nothing at or after the start: idle
    g = _run(conf, ent, am, tok, msk, bs, uni, B, L, BL, 0.5, 0)
    assert g[3][:3].tolist() == [-2, -2, -1]
    assert np.all(g[1][:3 * L] == 1) and np.all(g[4][:3] == 0) and np.all(g[5][:3] == -1)


@pytest.mark.parametrize("B", [1 << 16, 1 << 18])
@pytest.mark.parametrize("outputs", ["all", "none"])
def test_position_major_sweep_shape_matches_row_major(B, outputs):
    """The benchmark's sweep shape (blocks of 32 positions, one block per
    sequence, every sequence falling back), 2^16 sequences (one per lane)
    and 2^18 (four per lane): position-major and row-major give the same
    decisions, and every sequence commits its leftmost masked position."""
    _need_gpu()
    L, BL = 32, 32
    rng = np.random.default_rng(11)
    conf = (rng.random(B * L) * 0.03).astype(np.float32)
    am = rng.integers(0, 126464, B * L).astype(np.int32)
    tok = np.full(B * L, -1, np.int32)
    msk = np.ones(B * L, np.uint8)
    msk.reshape(B, L)[:, :5] = 0
    bs = np.zeros(B, np.int32)
    ent = np.zeros(B * L, np.float32)
    uni = np.zeros(B, np.float32)
    a = _run(conf, ent, am, tok, msk, bs, uni, B, L, BL, 0.9, 0, outputs=outputs)
    b = _run(conf, ent, am, tok, msk, bs, uni, B, L, BL, 0.9, 0,
             _binding.FORK_LAYOUT_POSITION_MAJOR, outputs=outputs)
    for x, y in zip(a, b):
        assert np.array_equal(x, y)
    assert np.all(a[3] == 1)
    if outputs == "all":
        assert np.all(a[5][:, 0] == 5) and np.all(a[5][:, 1:] == -1)
    assert np.array_equal(a[0].reshape(B, L)[:, 5], am.reshape(B, L)[:, 5])
    assert np.all(a[1].reshape(B, L)[:, :6] == 0) and np.all(a[1].reshape(B, L)[:, 6:] == 1)


@pytest.mark.parametrize("B,L,BL", [((1 << 18), 40, 32), ((1 << 18) + 2, 33, 16),
                                    ((1 << 18), 20, 20)])
@pytest.mark.parametrize("rule", [0, 1, 2, 3, 4])
@pytest.mark.parametrize("outputs", ["all", "ncommit", "none"])
def test_position_major_large_batches_match_row_major(B, L, BL, rule, outputs):
    """Batches large enough for four sequences per lane (and one not a
    multiple of four): random states, half of them sharing a block start,
    position-major against row-major (itself checked against the oracle).
    Without the commit positions, groups of four sequences that commit one
    position each, the same one, take the vector commit."""
    _need_gpu()
    conf, ent, am, tok, msk, bs, uni = _state(B, L, 1000, B + L + BL + rule)
    bs[: B // 2] = min(L - BL, 2)
    # a quarter of the sequences: one masked position, the same in each group
    # of four, so the vector commit runs for every rule
    q = B // 4
    msk.reshape(B, L)[:q] = 0
    msk.reshape(B, L)[:q, min(L - BL, 2) + 1] = 1
    for tau in (0.3, 0.9):
        a = _run(conf, ent, am, tok, msk, bs, uni, B, L, BL, tau, rule, outputs=outputs)
        b = _run(conf, ent, am, tok, msk, bs, uni, B, L, BL, tau, rule,
                 _binding.FORK_LAYOUT_POSITION_MAJOR, outputs=outputs)
        for k, (x, y) in enumerate(zip(a, b)):
            assert np.array_equal(x, y), k
        if outputs != "all":
            assert np.all(a[5] == -9) and (outputs == "ncommit" or np.all(a[4] == -9))
