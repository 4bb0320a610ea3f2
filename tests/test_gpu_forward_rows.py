"""Calls without a gradient over rows longer than one workgroup's registers:
whole and ragged packs, one and several chunks per row, chunks with fewer packs
than threads, waves in both forms within a row; against the oracle."""
import numpy as np
import pytest
import torch

from gpu_support import (check_loss, check_stats, check_token_kl, check_token_lse, ids_to_device, log)
from oracle import turnkl_oracle as O
from paper_2607_05804_amd import turnkl as T

pytestmark = pytest.mark.gpu


def _forward(zs, zt, dtype, vpt, ld=0, seed=0, start=0, ld_t=None, start_t=None):
    n, V = zs.shape
    rng = np.random.default_rng(seed)
    traj = (np.arange(n) // 12).astype(np.int32)
    turn = (np.arange(n) // 3 % 4).astype(np.int32)
    mask = (rng.random(n) < 0.7).astype(np.uint8)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    xs, xt = torch.from_numpy(zs).to(dt), torch.from_numpy(zt).to(dt)
    bits = (lambda x: x.view(torch.int16).numpy().view(np.uint16)) if dtype == "bf16" \
        else (lambda x: x.numpy())
    ref = O.fwd_bwd(traj, turn, mask, 0.4, 4, lambda r: (bits(xs)[r], bits(xt)[r]),
                    O.DTYPE_BF16 if dtype == "bf16" else O.DTYPE_F32)
    turn_d, traj_d, mask_d = ids_to_device(traj, turn, mask)

    def place(x, ld, start):
        if not ld:
            return x.cuda()
        buf = torch.full((start + n * ld,), 7.0, dtype=dt, device="cuda")[start:].view(n, ld)[:, :V]
        buf.copy_(x)
        return buf

    a = place(xs, ld, start)
    b = place(xt, ld if ld_t is None else ld_t, start if start_t is None else start_t)
    stats = T.new_turn_stats(4)
    lse = torch.empty((n, 2), dtype=torch.float32, device="cuda")
    T.set_row_tiling(vpt)
    try:
        outs = []
        for _ in range(3):
            loss, _, _, kl, _ = T.fwd_bwd(a, b, turn_d, traj_d, mask_d, 0.4, grad=None, max_turns=4,
                                          turn_stats=stats, token_kl=True, token_lse=lse)
            torch.cuda.synchronize()
            outs.append((loss.clone(), kl.clone(), lse.clone()))
    finally:
        T.set_row_tiling(0)
    for o in outs[1:]:  # the last workgroup of a row differs, the bits do not
        assert all(torch.equal(x.view(torch.int32), y.view(torch.int32)) for x, y in zip(o, outs[0]))
    check_loss(loss, ref.loss)
    check_token_kl(kl, ref.kl, mask)
    check_stats(stats, ref.stats)
    check_token_lse(lse, ref.lse, mask)


@pytest.mark.parametrize("V,dtype,vpt,ld,shift", [
    (16392, "bf16", 0, 0, 0.0), (51200, "bf16", 0, 0, 0.0), (51208, "bf16", 0, 0, 0.0),
    (151936, "bf16", 0, 0, 0.0), (151936, "f32", 0, 0, 0.0), (8196, "f32", 0, 0, 0.0),
    (4096, "bf16", 1, 0, 0.0),              # two chunks of one pack a thread
    (512, "bf16", 1, 0, 0.0),               # a chunk of one wave
    (40, "f32", 2, 0, 600.0),               # ten packs
    (16385, "bf16", 0, 0, 0.0), (50257, "bf16", 0, 50304, 0.0), (50257, "f32", 0, 0, 0.0),
    (45057, "bf16", 0, 45090, 0.0), (151937, "bf16", 0, 0, 0.0),
    (151936, "bf16", 0, 0, 3000.0), (50257, "f32", 0, 0, -5000.0), (50257, "bf16", 0, 50300, 900.0),
])
def test_forward(V, dtype, vpt, ld, shift, gpu):
    log(f"forward V={V} {dtype} vpt={vpt} ld={ld} shift={shift}")
    rng = np.random.default_rng(V + vpt)
    zs = rng.normal(0, 3, (25, V)) + shift
    zt = zs + rng.normal(0, 1, zs.shape) - 0.5 * shift
    _forward(zs, zt, dtype, vpt, ld, V)


@pytest.mark.parametrize("V,dtype,ld,start,ld_t,start_t", [
    (50257, "bf16", 50257, 0, 50304, 0), (50257, "bf16", 50300, 3, 50257, 11),
    (50257, "f32", 50259, 5, 50304, 2),
    (50176, "bf16", 50176, 0, 50180, 0),    # whole packs in one matrix only
    (50176, "f32", 50176, 0, 50176, 1),
    (16385, "bf16", 16400, 63, 16385, 1),
])
def test_matrices_at_their_own_starts_and_strides(V, dtype, ld, start, ld_t, start_t, gpu):
    log(f"forward V={V} {dtype} ld={ld}+{start} teacher {ld_t}+{start_t}")
    rng = np.random.default_rng(V + ld)
    zs = rng.normal(0, 3, (25, V))
    zs[5:8] += 500.0
    _forward(zs, zs + rng.normal(0, 1, zs.shape), dtype, 0, ld, V, start, ld_t, start_t)


@pytest.mark.parametrize("V,dtype", [(50176, "bf16"), (50257, "bf16"), (20001, "f32"), (120000, "f32")])
def test_waves_in_both_forms(V, dtype, gpu):
    """Spikes past the sampled references, in the student, the teacher or both,
    at the row's first and last elements and inside it."""
    log(f"forward, spikes, V={V} {dtype}")
    rng = np.random.default_rng(V)
    zs = rng.normal(0, 3, (24, V))
    zt = zs + rng.normal(0, 1, zs.shape)
    at = [0, V - 1, V // 2, 9000, V - 700, 8191]
    for r in range(24):
        k = at[r % len(at)]
        if r % 3 != 1:
            zs[r, k] += 350.0
        if r % 3 != 0:
            zt[r, k] += 340.0
    _forward(zs, zt, dtype, 0, 0, V)


@pytest.mark.parametrize("n", [40, 8200])
def test_a_workspace_after_a_call_with_a_gradient(n, gpu):
    """The rows' arrival counters start from zero whatever the last call left in
    the workspace (there: scaled weights), on both kinds of prologue."""
    log(f"forward after a gradient call n={n}")
    V = 51208  # two chunks
    g = torch.Generator(device="cuda").manual_seed(n)
    zs = torch.randn((n, V), generator=g, device="cuda").mul_(3).bfloat16()
    zt = torch.randn((n, V), generator=g, device="cuda").mul_(3).bfloat16()
    at = np.arange(n)
    ids = ids_to_device((at // 12).astype(np.int32), (at // 3 % 4).astype(np.int32),
                        (at % 5 != 0).astype(np.uint8))
    want = T.fwd_bwd(zs, zt, *ids, 0.4, grad=None, max_turns=4, token_kl=True)
    ws = T.Workspace(n, V, T.BF16, 4, aligned_rows=True)
    T.fwd_bwd(zs, zt, *ids, 0.4, grad="new", grad_scale=-2.5, max_turns=4, workspace=ws)
    for scale in (1.0, -3.0):
        loss, _, _, kl, _ = T.fwd_bwd(zs, zt, *ids, 0.4, grad=None, grad_scale=scale, max_turns=4,
                                      token_kl=True, workspace=ws)
        torch.cuda.synchronize()
        assert torch.equal(loss, want[0]) and torch.equal(kl, want[3])
