"""The dense gradient of the top-K call under every form of its zero-fill: rows
without padding (whole packs or not, any start), rows at a stride, rows
shorter than a pack, a single row; out of place and in place."""
import numpy as np
import pytest
import torch

from gpu_support import ids_to_device, log
from paper_2607_05804_amd import turnkl as T

pytestmark = pytest.mark.gpu

GUARD = 200


@pytest.mark.parametrize("n,V,pad,start,dtype", [
    (21, 4096, 0, 0, "bf16"),    # whole packs
    (21, 4097, 0, 0, "bf16"),    # an odd total: elements after the last pack
    (20, 1003, 0, 3, "bf16"),    # elements before the first pack, too
    (1, 777, 31, 5, "bf16"),     # one row
    (3, 5, 0, 1, "bf16"),        # fewer than two packs in all
    (21, 2048, 9, 0, "bf16"),    # rows at a stride, whole packs, off their lines
    (21, 2049, 62, 1, "bf16"),   # one element past a workgroup's packs
    (21, 16385, 62, 1, "bf16"),  # and past eight workgroups'
    (300, 40, 3, 1, "bf16"),     # many rows to a workgroup
    (200, 511, 2, 5, "bf16"),    # the longest rows on their own grid ...
    (200, 512, 2, 5, "bf16"),    # ... and the shortest on the lines'
    (1400, 151936, 1, 0, "bf16"),  # too large for default stores
    (40, 8, 3, 0, "bf16"),       # one pack a row
    (300, 7, 4, 1, "bf16"),      # rows shorter than a pack
    (21, 1001, 0, 1, "f32"),
    (21, 1025, 3, 2, "f32"),
    (30, 3, 2, 0, "f32"),
])
@pytest.mark.parametrize("mode", ["new", "inplace"])
def test_dense_gradient_is_the_support_gradient_and_zero(n, V, pad, start, dtype, mode, gpu):
    log(f"topk fill n={n} V={V} pad={pad} start={start} {dtype} {mode}")
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    rng = np.random.default_rng(n + V)
    k = min(V, 50)
    ids = torch.from_numpy(np.stack([rng.permutation(V)[:k] for _ in range(n)]).astype(np.int32)).cuda()
    vals = torch.from_numpy(rng.normal(0, 2, (n, k)).astype(np.float32)).cuda()
    mask = (rng.random(n) < 0.7).astype(np.uint8)
    mask[0] = 1
    turn_d, traj_d, mask_d = ids_to_device(np.zeros(n, np.int32), np.zeros(n, np.int32), mask)
    ld = V + pad
    flat = torch.full((GUARD + start + n * ld + GUARD,), 7.0, dtype=dt, device="cuda")
    g = flat[GUARD + start:GUARD + start + n * ld].view(n, ld)[:, :V]
    zs = torch.from_numpy(rng.normal(0, 2, (n, V)).astype(np.float32)).to(dt).cuda()
    if mode == "inplace":
        g.copy_(zs)
        zs = g
    _, out, gk, _, _, _ = T.fwd_bwd_topk(zs, ids, vals, turn_d, traj_d, mask_d, 0.5,
                                         grad="inplace" if mode == "inplace" else g, grad_topk=True,
                                         max_turns=1)
    torch.cuda.synchronize()
    want = torch.zeros((n, V), dtype=dt, device="cuda").scatter_(1, ids.long(), gk.to(dt))
    assert torch.equal(out.contiguous(), want)
    assert bool((gk != 0).any()) or k == 1
    rest = flat.clone()
    rest[GUARD + start:GUARD + start + n * ld].view(n, ld)[:, :V] = 7.0
    assert bool((rest == 7.0).all())
