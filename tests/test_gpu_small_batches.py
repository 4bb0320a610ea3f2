"""Segments and weights of small batches, which one workgroup computes: around
the sizes where the tokens per thread change and where the batch goes to the
tiled kernels, with up to a segment a token, and the earliest error in every
position; against the oracle."""
import numpy as np
import pytest
import torch

from gpu_support import check_loss, check_segments, check_stats, check_token_weights, ids_to_device, log
from oracle import turnkl_oracle as O
from paper_2607_05804_amd import turnkl as T

pytestmark = pytest.mark.gpu

V = 8
TURNS = 1024


def _batch(n, mean_len, seed, segments=None):
    """n tokens in turns of about mean_len tokens, up to 40 turns a trajectory,
    with padding between and inside trajectories' turns (and after the first
    `segments` segments; with more segments than tokens, no padding)."""
    rng = np.random.default_rng(seed)
    traj, turn = np.full(n, -1, np.int32), np.zeros(n, np.int32)
    i, b, t = 0, 0, 0
    while i < n:
        if rng.random() < 0.1 and not (segments or 0) > n:
            i += int(rng.integers(1, 3))  # padding
        k = int(rng.integers(1, 2 * mean_len)) if mean_len > 1 else 1
        traj[i:i + k], turn[i:i + k] = b, t
        i += k
        t += int(rng.integers(1, 3))
        if t >= 40 or rng.random() < 0.05:
            b, t = b + int(rng.integers(1, 4)), 0
    if segments is not None:
        start = (traj >= 0) & ((traj != np.roll(traj, 1)) | (turn != np.roll(turn, 1)))
        traj[np.cumsum(start) > segments] = -1
    mask = ((traj >= 0) & (rng.random(n) < 0.6)).astype(np.uint8)
    mask[traj == 3] = 0
    zs = rng.normal(0.0, 3.0, (n, V)).astype(np.float32)
    return traj, turn, mask, zs, (zs + rng.normal(0.0, 1.0, zs.shape)).astype(np.float32)


@pytest.mark.parametrize("n,mean_len,segments", [
    (1, 1, None), (63, 4, None), (1023, 30, None), (1024, 30, None), (1025, 30, None), (1025, 1, None),
    (4096, 20, None), (4097, 20, None), (3000, 2, None),
    (4096, 1, None), (8000, 3, None),                        # more than 2,048 segments
    (6000, 1, 4095), (6000, 1, 4096), (6000, 1, 4097), (6000, 1, 5000),
    (8000, 1, None), (8192, 1, None), (8192, 1, 1 << 20),    # the last without padding
    (8191, 40, None), (8192, 12, None), (8193, 12, None),    # the last goes to the tiled kernels
])
@pytest.mark.parametrize("floor,frac", [(0, 0.0), (2, 0.15)])
def test_segments_and_weights(n, mean_len, segments, floor, frac, gpu):
    log(f"small batch n={n} mean_len={mean_len} segments={segments} floor={floor}")
    traj, turn, mask, zs, zt = _batch(n, mean_len, n + mean_len, segments)
    turn_d, traj_d, mask_d = ids_to_device(traj, turn, mask)
    success = (traj % 2 == 0).astype(np.uint8)
    stats, ostats = T.new_turn_stats(TURNS), T.new_turn_stats(2 * TURNS)
    w = torch.empty(n, dtype=torch.float32, device="cuda")
    loss, _, _, kl, ws = T.fwd_bwd(
        torch.from_numpy(zs).cuda(), torch.from_numpy(zt).cuda(), turn_d, traj_d, mask_d, 0.3,
        grad=None, max_turns=TURNS, turn_stats=stats, token_weights=w, support_floor=floor,
        support_frac=frac, success=torch.from_numpy(success).cuda(), outcome_stats=ostats,
        token_kl=True)
    torch.cuda.synchronize()
    ref = O.fwd_bwd(traj, turn, mask, 0.3, TURNS, lambda r: (zs[r], zt[r]), O.DTYPE_F32,
                    support_floor=floor, support_frac=frac, success=success)
    assert ref.status == O.OK
    if segments is not None:
        assert ref.seg.count == min(segments, n)
    elif n >= 8000 and mean_len == 1:
        assert ref.seg.count > 6500
    check_segments(ws, ref.seg)
    check_token_weights(w, ref.w, mask)
    check_loss(loss, ref.loss)
    check_stats(stats, ref.stats)
    check_stats(ostats, ref.outcome_stats.reshape(-1))
    assert bool((kl[torch.from_numpy(mask).cuda() == 0] == 0).all())


@pytest.mark.parametrize("turns,floor", [(1, 0), (1, 1), (2048, 1), (8192, 0)])
def test_one_trajectory_of_8192_tokens(turns, floor, gpu):
    """The largest counts of the table, all supervised."""
    log(f"one trajectory, turns={turns} floor={floor}")
    n = 8192
    traj, turn, mask = np.zeros(n, np.int32), (np.arange(n) * turns // n).astype(np.int32), np.ones(n, np.uint8)
    rng = np.random.default_rng(turns)
    zs = rng.normal(0.0, 3.0, (n, V)).astype(np.float32)
    zt = (zs + rng.normal(0.0, 1.0, zs.shape)).astype(np.float32)
    stats = T.new_turn_stats(turns)
    w = torch.empty(n, dtype=torch.float32, device="cuda")
    loss, _, _, _, ws = T.fwd_bwd(torch.from_numpy(zs).cuda(), torch.from_numpy(zt).cuda(),
                                  *ids_to_device(traj, turn, mask), 0.3, grad=None, max_turns=turns,
                                  turn_stats=stats, token_weights=w, support_floor=floor)
    torch.cuda.synchronize()
    ref = O.fwd_bwd(traj, turn, mask, 0.3, turns, lambda r: (zs[r], zt[r]), O.DTYPE_F32,
                    support_floor=floor)
    check_segments(ws, ref.seg)
    check_token_weights(w, ref.w, mask)
    check_loss(loss, ref.loss)
    check_stats(stats, ref.stats)


@pytest.mark.parametrize("n,mean_len", [(1500, 20), (3000, 1), (8000, 1), (7000, 30), (8193, 30)])
@pytest.mark.parametrize("kind", ["pad_mask", "turn_high", "order", "outcome"])
def test_the_earliest_error_is_reported(n, mean_len, kind, gpu):
    log(f"small batch error n={n} mean_len={mean_len} {kind}")
    traj, turn, mask, zs, zt = _batch(n, mean_len, n)
    success = (traj % 2 == 0).astype(np.uint8)
    inner = np.nonzero((traj >= 0) & (np.arange(n) > n // 3) & (np.arange(n) < n - 2))[0]
    i, late = int(inner[0]), int(inner[-1])
    if kind == "pad_mask":
        traj[i], mask[i] = -1, 1
    elif kind == "turn_high":
        turn[i] = TURNS
    elif kind == "order":
        traj[i:] = np.where(traj[i:] >= 0, 0, -1)
    else:
        success[i] ^= 1
    if kind != "order":  # a later error, of the first rank
        traj[late], mask[late] = -1, 1
    ref = O.segments(traj, turn, mask, TURNS)
    want = O.fwd_bwd(traj, turn, mask, 0.3, TURNS, lambda r: (zs[r], zt[r]), O.DTYPE_F32,
                     success=success).status
    assert want != O.OK and (kind == "outcome" or ref.status == want)
    turn_d, traj_d, mask_d = ids_to_device(traj, turn, mask)
    loss, _, _, _, ws = T.fwd_bwd(
        torch.from_numpy(zs).cuda(), torch.from_numpy(zt).cuda(), turn_d, traj_d, mask_d, 0.3,
        grad=None, max_turns=TURNS, check=False, success=torch.from_numpy(success).cuda(),
        outcome_stats=T.new_turn_stats(2 * TURNS))
    assert ws.status() == want
    assert torch.isnan(loss).all()
