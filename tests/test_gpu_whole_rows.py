"""Rows with one workgroup each: whole packs around the sizes where the
workgroup and the packs per thread change, more rows than the chip holds at
once, a spike that the fast form cannot take; against the oracle."""
import numpy as np
import pytest
import torch

from gpu_support import check_grad_rows, check_loss, check_stats, check_token_kl, ids_to_device, log
from oracle import turnkl_oracle as O
from paper_2607_05804_amd import turnkl as T

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V,dtype,n,shift,grad", [
    (8, "bf16", 40, 0.0, "new"), (512, "bf16", 9000, 0.0, "inplace"), (520, "bf16", 40, 0.0, "new"),
    (4096, "bf16", 40, 0.0, "new"), (4096, "bf16", 40, 700.0, "inplace"),  # one wave, eight packs a lane
    (4104, "bf16", 40, 0.0, "inplace"), (4104, "bf16", 40, 700.0, "new"),  # 256 threads, three packs
    (16384, "bf16", 40, 0.0, "new"), (16392, "bf16", 40, 0.0, "new"),      # the longest; chunks
    (4, "f32", 40, 0.0, "new"), (2048, "f32", 40, 0.0, "inplace"), (2052, "f32", 40, 0.0, None),
    (8192, "f32", 40, -900.0, "new"), (8192, "f32", 40, 0.0, None), (8196, "f32", 40, 0.0, "new"),
])
def test_rows_with_a_workgroup_each(V, dtype, n, shift, grad, gpu):
    log(f"whole rows V={V} {dtype} n={n} shift={shift} {grad}")
    rng = np.random.default_rng(V + n)
    traj = (np.arange(n) // 20).astype(np.int32)
    turn = (np.arange(n) // 5 % 4).astype(np.int32)
    mask = (rng.random(n) < 0.6).astype(np.uint8)
    zs = rng.normal(0, 3, (n, V)) + shift
    zt = zs + rng.normal(0, 1, (n, V)) - 0.5 * shift
    zs[:, -1] += 300.0 * (np.arange(n) % 7 == 0)  # past the sampled reference
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    xs, xt = torch.from_numpy(zs).to(dt), torch.from_numpy(zt).to(dt)
    bits = (lambda x: x.view(torch.int16).numpy().view(np.uint16)) if dtype == "bf16" \
        else (lambda x: x.numpy())
    rows = list(range(n)) if n < 1000 else list(range(0, n, 97))
    ref = O.fwd_bwd(traj, turn, mask, 0.4, 4, lambda r: (bits(xs)[r], bits(xt)[r]),
                    O.DTYPE_BF16 if dtype == "bf16" else O.DTYPE_F32, 1.0, rows)
    turn_d, traj_d, mask_d = ids_to_device(traj, turn, mask)
    stats = T.new_turn_stats(4)
    g = torch.full_like(xs, 9.0).cuda() if grad == "new" else grad
    loss, out, _, kl, _ = T.fwd_bwd(xs.cuda(), xt.cuda(), turn_d, traj_d, mask_d, 0.4, grad=g,
                                    max_turns=4, turn_stats=stats, token_kl=True)
    torch.cuda.synchronize()
    check_loss(loss, ref.loss)
    check_token_kl(kl, ref.kl, mask)
    check_stats(stats, ref.stats)
    if grad is not None:
        check_grad_rows(out, ref, 1.0, rows, mask)
        assert bool((out[torch.from_numpy(mask).cuda() == 0] == 0).all())


@pytest.mark.parametrize("n,grad", [(19520, "new"), (19584, "new"), (19584, None)])
def test_either_side_of_a_large_batch(n, grad, gpu):
    """Rows of 2,048 packs: above 40 million packs (19,532 rows) with a gradient
    they take tickets; one row in 97 supervised, the others zeros."""
    log(f"large batch n={n} {grad}")
    V = 16384
    rng = np.random.default_rng(n)
    sup = np.arange(0, n, 97)
    traj, turn = (np.arange(n) // 2000).astype(np.int32), (np.arange(n) // 500 % 4).astype(np.int32)
    mask = np.zeros(n, np.uint8)
    mask[sup] = 1
    zs = np.zeros((n, V), np.uint16)
    zt = np.zeros((n, V), np.uint16)
    a = rng.normal(0, 3, (sup.size, V)).astype(np.float32)
    to_bits = lambda x: torch.from_numpy(x).bfloat16().view(torch.int16).numpy().view(np.uint16)
    zs[sup], zt[sup] = to_bits(a), to_bits(a + rng.normal(0, 1, a.shape).astype(np.float32))
    ref = O.fwd_bwd(traj, turn, mask, 0.4, 4, lambda r: (zs[r], zt[r]), O.DTYPE_BF16, 1.0, list(sup))
    dev = lambda x: torch.from_numpy(x.view(np.int16)).cuda().view(torch.bfloat16)
    out = torch.full((n, V), 9.0, dtype=torch.bfloat16, device="cuda") if grad else None
    loss, out, _, kl, _ = T.fwd_bwd(dev(zs), dev(zt), *ids_to_device(traj, turn, mask), 0.4, grad=out,
                                    max_turns=4, token_kl=True)
    torch.cuda.synchronize()
    check_loss(loss, ref.loss)
    check_token_kl(kl, ref.kl, mask)
    if grad:
        check_grad_rows(out, ref, 1.0, list(sup), mask)
        assert int(torch.count_nonzero(out).item()) == int(torch.count_nonzero(
            out.index_select(0, torch.from_numpy(sup).cuda())).item())
