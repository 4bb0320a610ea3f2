"""Rows with runs of very low logits (masked columns), and rows with logits so far
above the others that the sums against the sampled references come near the
largest float: every form of the row kernels, with and without a gradient;
against the oracle."""
import numpy as np
import pytest
import torch

from gpu_support import (check_loss, check_stats, check_token_kl, check_token_lse, ids_to_device,
                         log, rows_bits_to_host, rows_to_host)
from oracle import turnkl_oracle as O
from paper_2607_05804_amd import turnkl as T

pytestmark = pytest.mark.gpu

# vocabulary, dtype, row stride (0: packed), tiling override
FORMS = [
    (151936, "bf16", 0, 0),       # whole packs, three chunks
    (50176, "bf16", 0, 0),        # one chunk
    (50176, "f32", 0, 0),         # two chunks
    (4096, "bf16", 0, 1),         # two chunks of one pack a thread
    (50257, "bf16", 0, 0),        # ragged packs, two chunks
    (50257, "f32", 50304, 0),
    (16384, "bf16", 0, 0),        # one workgroup a row
    (9001, "bf16", 0, 0),
    (1001, "f32", 0, 0),          # one wave a row
    (4000, "bf16", 0, 0),
    (7, "bf16", 0, 0),            # one element per load
]


def _compare(zs, zt, dtype, ld, vpt):
    """Loss, statistics, per-token KL, log-partition functions and gradient of
    both kinds of call.  The gradient bound of gpu_support, with its absolute
    part in units of the row's KL where that is above one (the factor
    d - KL of an element is computed to that accuracy)."""
    n, V = zs.shape
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    traj = (np.arange(n) // 6).astype(np.int32)
    turn = (np.arange(n) // 2 % 3).astype(np.int32)
    mask = np.ones(n, np.uint8)
    a = torch.full((n, ld or V), 7.0, dtype=dt, device="cuda")[:, :V]
    b = torch.full((n, ld or V), 7.0, dtype=dt, device="cuda")[:, :V]
    a.copy_(torch.from_numpy(zs))
    b.copy_(torch.from_numpy(zt))
    ha, hb = rows_bits_to_host(a, np.arange(n)), rows_bits_to_host(b, np.arange(n))
    ref = O.fwd_bwd(traj, turn, mask, 0.4, 3, lambda r: (ha[r], hb[r]),
                    O.DTYPE_BF16 if dtype == "bf16" else O.DTYPE_F32, grad_rows=list(range(n)))
    assert np.isfinite(ref.kl).all()
    ids = ids_to_device(traj, turn, mask)
    for grad in (None, "new"):
        stats = T.new_turn_stats(3)
        lse = torch.empty((n, 2), dtype=torch.float32, device="cuda")
        T.set_row_tiling(vpt)
        try:
            loss, g, _, kl, _ = T.fwd_bwd(a, b, *ids, 0.4, grad=grad, max_turns=3, turn_stats=stats,
                                          token_kl=True, token_lse=lse)
        finally:
            T.set_row_tiling(0)
        torch.cuda.synchronize()
        check_token_kl(kl, ref.kl, mask)
        check_token_lse(lse, ref.lse, mask)
        check_loss(loss, ref.loss)
        check_stats(stats, ref.stats)
        if grad is None:
            continue
        G = rows_to_host(g, np.arange(n)).astype(np.float64)
        for r in range(n):
            err = np.abs(G[r] / ref.w[r] - ref.grads[r])
            unit = max(1.0, abs(ref.kl[r]))
            rel, absolute = (2.0 ** -8, 2e-5) if dtype == "bf16" else (1e-4, 2e-6)
            bad = np.nonzero(~(err <= rel * np.abs(ref.grads[r]) + absolute * unit))[0]
            assert bad.size == 0, (r, bad[:5], G[r][bad[:5]] / ref.w[r], ref.grads[r][bad[:5]])


@pytest.mark.parametrize("value", [-1e4, -1e9, -1e30, -1e38, "lowest"])
@pytest.mark.parametrize("V,dtype,ld,vpt", FORMS)
def test_masked_columns(V, dtype, ld, vpt, value, gpu):
    """Runs at the row's start, middle and end, runs over whole chunks, and a
    random 90% of the columns, in the student, the teacher, both, or the student
    and every other column of them in the teacher; the other logits around 0 or
    70.  (In the teacher alone to -1e30: below, the row's sum of p (a - b)
    before its division leaves the float range.)"""
    log(f"masked V={V} {dtype} ld={ld} vpt={vpt} value={value}")
    rng = np.random.default_rng(V)
    col = np.arange(V)
    runs = [col < V // 6, (col >= V // 3) & (col < V // 2), col >= V - V // 6, col < 0.55 * V,
            col >= 0.3 * V, rng.random(V) < 0.9]
    runs[5][V // 2] = False
    low = float(torch.finfo(torch.bfloat16 if dtype == "bf16" else torch.float32).min) \
        if value == "lowest" else value
    whose = ("student", "both", "half") + (("teacher",) if low >= -1e30 else ())
    zs, zt = [], []
    for run in runs:
        for who in whose:
            for shift in (0.0, 70.0):
                s = rng.normal(0, 3, V) + shift
                t = s + rng.normal(0, 1, V)
                if who != "teacher":
                    s[run] = low
                if who != "student":
                    t[run & (col % 2 == 0) if who == "half" else run] = low
                zs.append(s)
                zt.append(t)
    _compare(np.stack(zs), np.stack(zt), dtype, ld, vpt)


@pytest.mark.parametrize("V,dtype,ld,vpt", FORMS[:-1])
def test_sums_near_the_largest_float(V, dtype, ld, vpt, gpu):
    """Student logits 80 to 89 above the sampled references: the sum of
    2^(..) (a - b) leaves the float range before the sum of 2^(..) does, and
    sums that fit one by one overflow together."""
    log(f"spikes V={V} {dtype} ld={ld} vpt={vpt}")
    rng = np.random.default_rng(V)
    zs, zt = [], []
    for up in (80.0, 84.0, 85.0, 86.0, 87.0, 88.0, 88.5):
        s = rng.normal(0, 3, V)
        t = s + rng.normal(0, 1, V)
        s[int(0.7 * V)] = s[:2048].max() + up
        zs.append(s)
        zt.append(t)
        # the same value many times over, in every wave and chunk
        s = np.zeros(V)
        s[int(0.2 * V)::max(V // 40, 1)] = up
        zs += [s, s]
        zt += [rng.normal(0, 1, V), s + rng.normal(0, 1, V)]
    _compare(np.stack(zs), np.stack(zt), dtype, ld, vpt)
