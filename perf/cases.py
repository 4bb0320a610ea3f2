"""Cases of the fused turn-KL calls whose time is measured.

A training or probe step hands the library the packed logits of a batch of
multi-turn agent trajectories and takes back the loss, the gradient of the
student logits (or of their top-K support) and the per-turn statistics.  The
listed cases are the batches of the repository's own workloads and benchmark,
plus the calls around them: micro-batches in place without a workspace,
forward-only probes, vocabularies that are no multiple of a 16-byte pack, fp32
logits and the top-K loss.  The 131,072-token stress batch is left out: three
of it do not fit the card beside their checks.

Inputs are drawn on the GPU from the seed: student logits N(0, 3^2), teacher =
student + noise that decays with the turn, optionally with a few boosted
columns per row, in the structure that the synthetic workloads use
(trajectories of turns, each an observation span followed by a supervised
response).
"""
import math

import numpy as np
import torch

from paper_2607_05804_amd import turnkl as T

ALPHA = 0.5
BLOCK = 1 << 28  # elements drawn at a time
EXACT_GRAD_BYTES = 6 << 30  # larger float64 gradients are not formed


def _case(name, kind, tokens, vocab, dtype="bf16", trajs=8, turns=10, masked=0.4, peaks=0,
          pad_cols=0, pad_rows=0, k=0):
    """kind: "fused" (gradient out of place), "inplace" (over the student
    logits, built-in scratch, statistics accumulated), "forward" (no gradient;
    support floor, outcome statistics and log-partition functions), "topk"
    (dense gradient) or "topk_sparse" (gradient on the support).  masked: the
    observation share of each turn.  peaks: boosted columns per row.
    pad_cols: columns between the vocabulary and the row stride.  pad_rows:
    padding tokens at the end of the batch."""
    return {"name": name, "kind": kind, "tokens": tokens, "vocab": vocab, "dtype": dtype,
            "trajs": trajs, "turns": turns, "masked": masked, "peaks": peaks, "pad_cols": pad_cols,
            "pad_rows": pad_rows, "k": k}


def listed():
    return [
        # a unit-test or toy-vocabulary step: launches and latency
        _case("tiny_fp32", "fused", 160, 1024, "f32", trajs=2, turns=4, masked=0.0),
        # a small agent step over a 32,000-entry vocabulary
        _case("agent", "fused", 4166, 32000, trajs=8, turns=10),
        # one trajectory of an accumulated step, gradient over its logits, no allocation
        _case("micro_inplace", "inplace", 1500, 151936, trajs=1, turns=30),
        # a step of short turns, mostly observations, with peaked distributions
        _case("peaked", "fused", 16534, 151936, trajs=16, turns=30, masked=0.6, peaks=5,
              pad_rows=42),
        # the benchmark's long-horizon step
        _case("long_horizon", "fused", 65536, 151936, trajs=30, turns=50),
        # a batch packed from response tokens only
        _case("responses_only", "fused", 8192, 151936, trajs=16, turns=20, masked=0.0),
        # a model that keeps its logits in fp32
        _case("fp32_logits", "fused", 4096, 151936, "f32", trajs=8, turns=16),
        # a depth-controller probe: losses, statistics and outcome split, no gradient
        _case("probe_forward", "forward", 16384, 151936, trajs=32, turns=40),
        # a 50,257-entry vocabulary, rows packed without padding
        _case("ragged_vocab", "fused", 6000, 50257, trajs=8, turns=12),
        # the same vocabulary cut from logits padded to 50,304 columns, fp32
        _case("padded_stride_fp32", "fused", 3000, 50257, "f32", trajs=8, turns=12, pad_cols=47),
        # the teacher's top-50 support, dense gradient
        _case("topk_dense", "topk", 16384, 151936, trajs=16, turns=30, k=50),
        # the same loss for a caller that scatters the support gradient itself
        _case("topk_sparse", "topk_sparse", 65536, 151936, trajs=30, turns=50, k=50),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["fused", "fused", "fused", "fused", "inplace", "forward", "forward", "topk",
                       "topk_sparse"])
    dtype = rng.choice(["bf16", "bf16", "bf16", "f32"])
    es = 2 if dtype == "bf16" else 4
    vocab = _log_int(rng, 1000, 160000)
    form = rng.choice(["any", "any", "eight", "sixtyfour"])
    if form == "eight":
        vocab -= vocab % 8
    elif form == "sixtyfour":
        vocab += -vocab % 64
    pad_cols = rng.choice([0, 0, 0, -vocab % 64, rng.randrange(1, 100)])
    # 12 GB of the three matrices at most; the built-in scratch holds 16,384
    # tokens of any of these vocabularies
    most = min(65536, int(12e9 / (3 * es * vocab)))
    if kind == "inplace":
        most = min(most, 16384)
    tokens = _log_int(rng, 64, most)
    trajs = max(1, min(64, _log_int(rng, 1, max(1, tokens // 16))))
    turns = max(1, min(50, tokens // (8 * trajs)))
    turns = rng.randrange(1, turns + 1)
    return {"kind": kind, "tokens": tokens, "vocab": vocab, "dtype": dtype, "trajs": trajs,
            "turns": turns, "masked": rng.choice([0.0, 0.2, 0.4, 0.6]),
            "peaks": rng.choice([0, 0, 5]), "pad_cols": pad_cols,
            "pad_rows": rng.choice([0, 0, tokens % 64]),
            "k": _log_int(rng, 1, 128) if kind.startswith("topk") else 0}


# ---------------------------------------------------------------------------
# inputs


def _structure(case, seed):
    """Trajectory ids, turn ids and loss mask (numpy), padding last."""
    rng = np.random.default_rng(seed)
    n, b = case["tokens"], case["trajs"]
    counts = rng.integers((case["turns"] + 1) // 2, case["turns"] + 1, size=b)
    counts[0] = case["turns"]
    n_seg = int(counts.sum())
    share = rng.lognormal(0.0, 0.6, size=n_seg)
    # every turn at least one token, the rest by share
    cuts = np.floor(np.cumsum(share) / share.sum() * (n - n_seg) + 0.5).astype(np.int64)
    lens = np.diff(np.concatenate([[0], cuts])) + 1
    lens[-1] += n - int(lens.sum())
    traj = np.repeat(np.repeat(np.arange(b), counts), lens)
    turn_of = np.concatenate([np.arange(c) for c in counts])
    turn = np.repeat(turn_of, lens)
    start = np.repeat(np.cumsum(lens) - lens, lens)
    observed = np.repeat(np.floor(case["masked"] * lens + 0.5).astype(np.int64), lens)
    mask = (np.arange(n) - start) >= observed
    pad = case["pad_rows"]
    traj = np.concatenate([traj, np.full(pad, -1)])
    turn = np.concatenate([turn, np.zeros(pad, np.int64)])
    mask = np.concatenate([mask, np.zeros(pad, bool)])
    return traj.astype(np.int32), turn.astype(np.int32), mask.astype(np.uint8)


def _matrix(case):
    n, ld = case["tokens"] + case["pad_rows"], case["vocab"] + case["pad_cols"]
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    return torch.empty((n, ld), dtype=dt, device="cuda")[:, :case["vocab"]]


def _logits(case, seed, turn):
    g = torch.Generator(device="cuda").manual_seed(seed * 2 + 1)
    zs, zt = _matrix(case), _matrix(case)
    n, v = zs.shape
    sigma = (1.5 * 0.95 ** turn.double()).float()[:, None]
    step = max(1, BLOCK // v)
    for r in range(0, n, step):
        a = torch.randn((min(step, n - r), v), generator=g, device="cuda").mul_(3.0)
        if case["peaks"]:
            at = torch.randint(0, v, (a.shape[0], case["peaks"]), generator=g, device="cuda")
            a.scatter_add_(1, at, torch.full(at.shape, 10.0, device="cuda"))
        zs[r:r + step] = a
        a += torch.randn(a.shape, generator=g, device="cuda").mul_(sigma[r:r + step])
        zt[r:r + step] = a
    return zs, zt


def _support(case, seed, n):
    """Distinct ids spread over the vocabulary and descending teacher values."""
    g = torch.Generator(device="cuda").manual_seed(seed * 2 + 2)
    k, v = case["k"], case["vocab"]
    u = torch.rand((n, k), generator=g, device="cuda")
    edge = torch.arange(k, device="cuda") * v // k
    width = (torch.arange(1, k + 1, device="cuda") * v // k) - edge
    ids = edge + torch.minimum((u * width).long(), width - 1)
    ids = ids.gather(1, torch.rand((n, k), generator=g, device="cuda").argsort(1))
    vals = torch.randn((n, k), generator=g, device="cuda").abs_().mul_(1.5).add_(10.0)
    return ids.int().contiguous(), vals.sort(1, descending=True).values.contiguous()


def _stat_views(buf):
    """The whole-number and the float columns of a statistics buffer."""
    return (buf.view(torch.int64).view(-1, T.STAT_FIELDS)[:, :2],
            buf.view(torch.float64).view(-1, T.STAT_FIELDS)[:, 2:])


def _inputs(case, seed):
    traj, turn, mask = _structure(case, seed)
    s = {"traj_np": traj, "turn_np": turn, "mask_np": mask}
    s["traj"], s["turn"], s["mask"] = (torch.from_numpy(x).cuda() for x in (traj, turn, mask))
    if case["kind"].startswith("topk"):
        n = traj.shape[0]
        g = torch.Generator(device="cuda").manual_seed(seed * 2 + 1)
        s["ids"], s["vals"] = _support(case, seed, n)
        s["zs"] = _matrix(case)
        step = max(1, BLOCK // case["vocab"])
        for r in range(0, n, step):
            a = torch.randn((min(step, n - r), case["vocab"]), generator=g, device="cuda").mul_(3.0)
            near = s["vals"][r:r + step]
            near = near + torch.randn(near.shape, generator=g, device="cuda")
            s["zs"][r:r + step] = a.scatter_(1, s["ids"][r:r + step].long(), near)
    else:
        s["zs"], s["zt"] = _logits(case, seed, s["turn"])
    if case["kind"] == "forward":
        s["success"] = (s["traj"] % 2 == 0).to(torch.uint8)
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    kind, n, turns = case["kind"], s["traj"].shape[0], case["turns"]
    s["kind"] = kind
    s["max_turns"] = turns
    s["stats"] = T.new_turn_stats(turns)
    s["counts"], s["moments"] = _stat_views(s["stats"])
    s["kl"] = torch.empty(n, dtype=torch.float32, device="cuda")
    dt = T.BF16 if case["dtype"] == "bf16" else T.F32
    es = 2 if case["dtype"] == "bf16" else 4
    ld = case["vocab"] + case["pad_cols"]
    if kind in ("fused", "forward"):
        s["ws"] = T.Workspace(n, case["vocab"], dt, turns, aligned_rows=ld * es % 16 == 0)
    elif kind.startswith("topk"):
        s["ws"] = T.TopkWorkspace(n, case["k"], turns)
    if kind in ("fused", "topk"):
        s["grad"] = _matrix(case)
    if kind == "inplace":
        s["loss"] = torch.empty(3, dtype=torch.float32, device="cuda")
        s["status"] = torch.empty(1, dtype=torch.int32, device="cuda")
    if kind == "forward":
        s["ostats"] = T.new_turn_stats(2 * turns)
        s["ocounts"], s["omoments"] = _stat_views(s["ostats"])
        s["lse"] = torch.empty((n, 2), dtype=torch.float32, device="cuda")
    if kind == "topk_sparse":
        s["grad_topk"] = torch.empty((n, case["k"]), dtype=torch.float32, device="cuda")
    return s


def run(s):
    kind = s["kind"]
    if kind == "inplace":
        T.fwd_bwd_noalloc(s["zs"], s["zt"], s["turn"], s["traj"], s["mask"], ALPHA, s["loss"],
                          grad="inplace", max_turns=s["max_turns"], turn_stats=s["stats"],
                          accumulate_stats=True, token_kl=s["kl"], status=s["status"])
        return {"loss": s["loss"], "grad": s["zs"], "kl": s["kl"], "counts": s["counts"],
                "moments": s["moments"], "status": s["status"]}
    if kind == "fused":
        loss = T.fwd_bwd(s["zs"], s["zt"], s["turn"], s["traj"], s["mask"], ALPHA, grad=s["grad"],
                         max_turns=s["max_turns"], turn_stats=s["stats"], token_kl=s["kl"],
                         workspace=s["ws"], check=False)[0]
        return {"loss": loss, "grad": s["grad"], "kl": s["kl"], "counts": s["counts"],
                "moments": s["moments"]}
    if kind == "forward":
        loss = T.fwd_bwd(s["zs"], s["zt"], s["turn"], s["traj"], s["mask"], ALPHA, grad=None,
                         max_turns=s["max_turns"], turn_stats=s["stats"], token_kl=s["kl"],
                         workspace=s["ws"], check=False, support_floor=8, support_frac=0.15,
                         success=s["success"], outcome_stats=s["ostats"], token_lse=s["lse"])[0]
        return {"loss": loss, "kl": s["kl"], "lse": s["lse"], "counts": s["counts"],
                "moments": s["moments"], "ocounts": s["ocounts"], "omoments": s["omoments"]}
    sparse = kind == "topk_sparse"
    loss = T.fwd_bwd_topk(s["zs"], s["ids"], s["vals"], s["turn"], s["traj"], s["mask"], ALPHA,
                          grad=None if sparse else s["grad"],
                          grad_topk=s["grad_topk"] if sparse else False,
                          max_turns=s["max_turns"], turn_stats=s["stats"], token_kl=s["kl"],
                          workspace=s["ws"], check=False)[0]
    return {"loss": loss, "grad": s["grad_topk"] if sparse else s["grad"], "kl": s["kl"],
            "counts": s["counts"], "moments": s["moments"]}


def work(case):
    n = case["tokens"] + case["pad_rows"]
    sup = int(round(case["tokens"] * (1.0 - case["masked"])))
    es = 2 if case["dtype"] == "bf16" else 4
    row = case["vocab"] * es
    support = sup * case["k"] * (4 + 4 + es)
    by = {"fused": (n + 2 * sup) * row, "inplace": (n + 2 * sup) * row, "forward": 2 * sup * row,
          "topk": n * row + support, "topk_sparse": support + n * case["k"] * 4}[case["kind"]]
    each = case["k"] if case["kind"].startswith("topk") else case["vocab"]
    return {"bytes": by + 13 * n, "flops": 20 * sup * each}


def tolerance(case):
    # About four times the largest error against exact(): 1.8e-3 for a bf16
    # gradient (its rounding), 1.0e-6 for fp32 outputs.
    if case["dtype"] == "bf16" and case["kind"] in ("fused", "inplace", "topk"):
        return {"rel": 7e-3, "max": 2e-2}
    return {"rel": 5e-6, "max": 2e-4}


# ---------------------------------------------------------------------------
# the same in 64 bits


def _rows64(a, b):
    """KL, its gradient and both log-partition functions of some rows."""
    la, lb = a.logsumexp(1, keepdim=True), b.logsumexp(1, keepdim=True)
    p = (a - la).exp()
    d = (a - la) - (b - lb)
    kl = (p * d).sum(1, keepdim=True)
    return kl[:, 0], p * (d - kl), torch.cat([la, lb], 1)


def _weights64(case, traj, turn, mask, floor, frac):
    """Per-token (w, w_traj, w_turn) of the blended, trajectory and turn means."""
    n, turns = traj.shape[0], case["turns"]
    on = mask > 0
    b_ids = np.unique(traj[on])
    b = len(b_ids)
    surv = np.array([len(np.unique(traj[on & (turn == t)])) for t in range(turns)])
    n_min = max(floor, math.ceil(frac * b))
    w_traj, w_turn = np.zeros(n), np.zeros(n)
    for i in b_ids:
        of = on & (traj == i)
        w_traj[of] = 1.0 / (b * of.sum())
        valid = [t for t in np.unique(turn[of]) if surv[t] >= n_min]
        for t in valid:
            at = of & (turn == t)
            w_turn[at] = 1.0 / (b * len(valid) * at.sum())
        if not valid:
            w_turn[of] = w_traj[of]
    return (1.0 - ALPHA) * w_traj + ALPHA * w_turn, w_traj, w_turn


def _stats64(traj, turn, on, kl, w, turns):
    out = np.zeros((turns, 4))
    for t in range(turns):
        at = on & (turn == t)
        if at.any():
            x = kl[at]
            m2 = float(((x - x.mean()) ** 2).sum())
            out[t] = [x.mean(), m2, m2 / x.size, float((w[at] * x).sum())]
    return out


def exact(case, seed):
    s = _inputs(case, seed)
    kind = case["kind"]
    traj, turn, mask = s["traj_np"], s["turn_np"], s["mask_np"]
    n, v = traj.shape[0], case["vocab"]
    floor, frac = (8, 0.15) if kind == "forward" else (0, 0.0)
    w, w_traj, w_turn = _weights64(case, traj, turn, mask, floor, frac)
    cols = case["k"] if kind == "topk_sparse" else v
    keep = kind != "forward" and n * cols * 8 <= EXACT_GRAD_BYTES
    grad = torch.zeros((n, cols), dtype=torch.float64, device="cuda") if keep else None
    kl = torch.zeros(n, dtype=torch.float64, device="cuda")
    lse = torch.full((n, 2), math.nan, dtype=torch.float64, device="cuda")
    on = np.nonzero(mask)[0]
    wd = torch.from_numpy(w).cuda()
    each = max(1, (1 << 26) // (case["k"] or v))
    for r in range(0, on.size, each):
        at = torch.from_numpy(on[r:r + each]).cuda()
        if case["k"]:
            ids = s["ids"][at].long()
            a, b = s["zs"][at[:, None], ids].double(), s["vals"][at].double()
        else:
            a, b = s["zs"][at].double(), s["zt"][at].double()
        kl[at], g, lse[at] = _rows64(a, b)
        if keep:
            g *= wd[at][:, None]
            if kind == "topk":
                grad[at[:, None], ids] = g
            else:
                grad[at] = g
    klh = kl.cpu().numpy()
    loss = np.array([(x * klh).sum() for x in (w, w_traj, w_turn)])
    sup = mask > 0
    out = {"loss": loss, "kl": kl, "counts": None,
           "moments": _stats64(traj, turn, sup, klh, w, case["turns"])}
    if kind == "forward":
        good = traj % 2 == 0
        out["lse"] = lse
        out["ocounts"] = None
        out["omoments"] = np.concatenate([_stats64(traj, turn, sup & f, klh, w, case["turns"])
                                          for f in (~good, good)])
    else:
        out["grad"] = grad
    if kind == "inplace":
        out["status"] = None
    return out
