"""Rows of any start and length on the 16-byte path: rows packed without
padding, matrices whose rows start at different places within a cache line,
the sizes around a pack, a wave of packs and a chunk, in place and with the
references subtracted per element."""
import numpy as np
import pytest
import torch

from gpu_support import (check_grad_rows, check_loss, check_stats, check_token_kl, ids_to_device,
                         log)
from oracle import turnkl_oracle as O
from paper_2607_05804_amd import turnkl as T

pytestmark = pytest.mark.gpu

GUARD = 173  # elements around the rows, which no call may write


def _place(x, ld, start):
    """The rows of x at stride ld, `start` elements into a guarded buffer."""
    n, v = x.shape
    flat = torch.full((GUARD + start + n * ld + GUARD,), 7.0, dtype=x.dtype, device=x.device)
    view = flat[GUARD + start:GUARD + start + n * ld].view(n, ld)[:, :v]
    view.copy_(x)
    return flat, view


def _rest_untouched(flat, view, start):
    n, v = view.shape
    ld = view.stride(0)
    f = flat.clone()
    f[GUARD + start:GUARD + start + n * ld].view(n, ld)[:, :v] = 7.0
    return bool((f == 7.0).all())


# vocabulary, dtype, (start, ld - V) of student, teacher and gradient, mode,
# common offset of the logits
CASES = [
    (8, "bf16", (0, 0), (0, 0), (0, 0), "new", 0.0),          # one pack, rows at every 16 bytes
    (9, "bf16", (0, 0), (1, 2), (3, 0), "new", 0.0),          # two packs over one another
    (15, "bf16", (5, 0), (5, 0), (5, 0), "inplace", 0.0),
    (4, "f32", (1, 0), (0, 1), (2, 3), "new", 0.0),
    (7, "f32", (0, 0), (0, 0), (0, 0), "inplace", 0.0),
    (2041, "bf16", (0, 0), (0, 0), (0, 0), "new", 0.0),       # 256 packs or one more, by the row's start
    (2049, "bf16", (0, 63), (0, 63), (0, 63), "new", 0.0),    # one element past 256 packs, rows on lines
    (4097, "bf16", (2, 0), (0, 5), (1, 7), "new", 0.0),
    (1001, "f32", (0, 0), (0, 0), (0, 0), "forward", 0.0),
    (4030, "bf16", (0, 0), (1, 0), (0, 0), "new", 0.0),       # one wave or 256 threads, by the row's start
    (2023, "f32", (3, 0), (3, 0), (3, 0), "inplace", 800.0),
    (16319, "bf16", (0, 0), (0, 0), (5, 0), "new", 0.0),      # the longest rows with a workgroup each
    (16321, "bf16", (0, 0), (0, 0), (5, 0), "inplace", 0.0),  # chunks
    (45057, "bf16", (0, 0), (0, 0), (0, 0), "inplace", 0.0),  # one element past the widest chunk
    (50257, "bf16", (0, 0), (0, 0), (0, 0), "new", 0.0),
    (50257, "f32", (0, 47), (0, 47), (0, 47), "new", 0.0),
    (151937, "bf16", (0, 0), (0, 0), (0, 0), "inplace", 0.0),
    (151936, "bf16", (1, 0), (1, 0), (1, 0), "new", 0.0),     # whole packs, rows off them
    (4099, "bf16", (0, 0), (0, 0), (0, 0), "inplace", 900.0),  # offset rows
    (50257, "f32", (3, 1), (3, 1), (3, 1), "inplace", -5000.0),
    (50257, "bf16", (0, 0), (0, 0), (0, 0), "new", 3000.0),
]


@pytest.mark.parametrize("V,dtype,at_s,at_t,at_g,mode,shift", CASES)
def test_rows_of_any_start_and_length(V, dtype, at_s, at_t, at_g, mode, shift, gpu):
    log(f"ragged rows V={V} {dtype} {at_s} {at_t} {at_g} {mode} shift={shift}")
    rng = np.random.default_rng(V + int(abs(shift)))
    traj = np.repeat(np.arange(3), 9).astype(np.int32)
    turn = np.tile(np.repeat(np.arange(3), 3), 3).astype(np.int32)
    mask = (rng.random(27) < 0.7).astype(np.uint8)
    zs = rng.normal(0, 3, (27, V)) + shift
    zt = zs + rng.normal(0, 1, (27, V)) - 0.5 * shift
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    xs = torch.from_numpy(zs).to(dt)
    xt = torch.from_numpy(zt).to(dt)
    bits = (lambda x: x.view(torch.int16).numpy().view(np.uint16)) if dtype == "bf16" \
        else (lambda x: x.numpy())
    ref = O.fwd_bwd(traj, turn, mask, 0.3, 3, lambda r: (bits(xs)[r], bits(xt)[r]),
                    O.DTYPE_BF16 if dtype == "bf16" else O.DTYPE_F32, 1.0, list(range(27)))
    fs, s = _place(xs.cuda(), V + at_s[1], at_s[0])
    ft, t = _place(xt.cuda(), V + at_t[1], at_t[0])
    fg, g = _place(torch.zeros_like(xs).cuda(), V + at_g[1], at_g[0])
    turn_d, traj_d, mask_d = ids_to_device(traj, turn, mask)
    stats = T.new_turn_stats(3)
    grad = {"new": g, "inplace": "inplace", "forward": None}[mode]
    loss, out, _, kl, _ = T.fwd_bwd(s, t, turn_d, traj_d, mask_d, 0.3, grad=grad, max_turns=3,
                                    turn_stats=stats, token_kl=True)
    torch.cuda.synchronize()
    check_loss(loss, ref.loss)
    check_token_kl(kl, ref.kl, mask)
    check_stats(stats, ref.stats)
    if mode != "forward":
        check_grad_rows(out, ref, 1.0, range(27), mask)
    assert _rest_untouched(ft, t, at_t[0])
    assert _rest_untouched(fs, s, at_s[0])
    assert _rest_untouched(fg, g, at_g[0])
    if mode != "inplace":
        assert torch.equal(s.cpu(), xs)
    assert torch.equal(t.cpu(), xt)
