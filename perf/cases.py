"""Performance cases of the parameter-sync path: one GPU's shard, through the
package's entry points.

A case names an entry point ("kind"), how the shard is cut into segments
("segs") and the shape of the round: R peer gradients, G federation groups, A
local steps, H replicas of the sharding group.  listed() holds the cases by
what they stand for in a training run; draw() gives more of the same ranges.

Segment forms: "flat" (one segment), "ragged" (n elements cut at nseg - 1
random places), "model" (the Llama-3.1-8B shard of a rank in a sharding group
of S) and "layer" (one decoder layer of it, the unit FSDP wraps).

Values are those of a run in progress: master N(0, 0.02), gradients N(0, 1e-3)
or Student-t(3) with zeros, m and v at the size such gradients give them,
replicas near the own shard, step numbers past the warm-up.
"""
import numpy as np
import torch

import paper_2609_20359_amd as P

ADAMW = dict(lr=3e-4, beta1=0.9, beta2=0.95, eps=1e-8, weight_decay=0.1)
OUTER = dict(lr=0.7, momentum=0.9, nesterov=True)
STEP0 = 101
SCHEDULE = (2000, 200)   # total steps, warm-up steps
VOCAB, HIDDEN, LAYERS, MLP, KV = 128256, 4096, 32, 14336, 1024
CHUNK = 1 << 25

ROUNDS = ("round", "round_noalloc", "round_outer", "round_hsdp", "round_hsdp_recv")

_BASE = dict(kind="round", segs="flat", n=0, S=0, nseg=1, R=1, G=1, A=1, H=1, sumsq=False,
             clip=0.0, scratch=False, reuse=False, heavy_tails=False)


def _case(**kw):
    return dict(_BASE, **kw)


def listed():
    return [
        # The smallest round: a 1 Mi-parameter model, launches and latency.
        _case(name="round_tiny", n=1 << 20, R=4, G=2, A=4, sumsq=True),
        # The benchmark: a Llama-3.1-8B rank in a sharding group of 8.
        _case(name="round_8b_s8", segs="model", S=8, R=8, G=4, A=8, sumsq=True, reuse=True),
        # The same model spread over 64 ranks: the most peers, from a caller
        # that must not allocate.
        _case(name="round_8b_s64", kind="round_noalloc", segs="model", S=64, R=64, G=8, A=2,
              sumsq=True, reuse=True),
        # FL+HSDP: four replicas of a sharding group of 16, the FedAvg member.
        _case(name="hsdp_member_s16", kind="round_hsdp", segs="model", S=16, R=16, G=4, A=4, H=4,
              sumsq=True, reuse=True),
        # FL+HSDP: the replica that receives the broadcast, on a small shard
        # whose norm segments are 32 elements.
        _case(name="hsdp_receiver_s128", kind="round_hsdp_recv", segs="model", S=128, R=8, G=4,
              A=4, H=2, sumsq=True, reuse=True),
        # One local step and the outer Nesterov step over eight groups.
        _case(name="outer_250m", kind="round_outer", n=250_000_000, R=4, G=8, A=1),
        # Many odd-sized segments, heavy-tailed gradients, clipped by reading
        # the gradients twice, with a learning-rate schedule.
        _case(name="clip_ragged_65m", segs="ragged", n=65_365_214, nseg=1000, R=16, G=16, A=4,
              sumsq=True, clip=1.0, reuse=True, heavy_tails=True),
        # Clipped with the gradient scratch, 32 ranks.
        _case(name="clip_scratch_s32", segs="model", S=32, R=32, G=4, A=2, sumsq=True, clip=1.0,
              scratch=True, reuse=True),
        # One decoder layer's step as its reduce-scatter completes.
        _case(name="step_layer_s8", kind="step", segs="layer", S=8, R=8, sumsq=True),
        # The clipped step of a multi-GPU caller (sum of squares, then the
        # step) on a small odd shard of three ranks.
        _case(name="step_clipped_1m", kind="step_clipped", segs="ragged", n=1_000_003, nseg=24,
              R=3, sumsq=True, clip=1.0),
        # The unfused chain (reduction, then AdamW) on a layer of 64 ranks.
        _case(name="reduce_adamw_s64", kind="reduce_adamw", segs="layer", S=64, R=6, sumsq=True),
        # FedAvg alone over an odd number of groups.
        _case(name="fedavg_50m", kind="fedavg", n=50_000_017, G=5),
    ]


MAX_BYTES = 100e9         # of a drawn pass
MAX_STATE = 24e9          # of a drawn case's arrays


def draw(rng):
    while True:
        c = dict(_BASE)
        c["kind"] = rng.choice(["round", "round", "round_noalloc", "round_outer", "round_hsdp",
                                "round_hsdp_recv", "step", "step", "step_clipped",
                                "reduce_adamw", "reduce_wire", "fedavg", "fedopt", "recv"])
        c["segs"] = rng.choice(["flat", "ragged", "ragged", "model", "layer"])
        if c["segs"] in ("model", "layer"):
            c["S"] = rng.choice([4, 8, 16, 32, 64, 128, 256, 512])
            if c["segs"] == "model" and c["S"] > 64:
                c["S"] = rng.choice([128, 256])   # the vocabulary divides no further
            c["nseg"] = 0
        else:
            c["n"] = int(2 ** rng.uniform(12, 29.9)) | rng.choice([0, 1, 3])
            if c["segs"] == "ragged":
                c["nseg"] = max(2, int(min(2000, c["n"] // 64, 2 ** rng.uniform(1, 11))))
        c["R"] = rng.choice([1, 2, 3, 4, 4, 5, 6, 8, 8, 12, 16, 16, 24, 32, 64])
        c["G"] = rng.choice([1, 2, 3, 4, 4, 5, 6, 8, 12, 16])
        if c["kind"] in ROUNDS:
            c["A"] = rng.choice([1, 2, 4, 8])
            c["reuse"] = rng.random() < 0.7
            c["clip"] = rng.choice([0.0, 0.0, 1.0])
            c["scratch"] = c["clip"] > 0 and rng.random() < 0.5
        if c["kind"] == "step_clipped":
            c["clip"] = 1.0
        if c["kind"].startswith("round_hsdp"):
            c["H"] = rng.choice([2, 2, 3, 4, 8])
        c["sumsq"] = (c["kind"] not in ("reduce_wire", "fedavg", "fedopt", "recv")
                      and rng.random() < 0.7)
        c["heavy_tails"] = rng.random() < 0.25
        if work(c)["bytes"] <= MAX_BYTES and _state_bytes(c) <= MAX_STATE:
            return c


# ---- shapes ----------------------------------------------------------------


def _segments(case):
    """(offsets, decay flags) of the case's shard."""
    if case["segs"] == "flat":
        return np.array([0, case["n"]], np.int64), np.ones(1, np.uint8)
    if case["segs"] == "ragged":
        rs = np.random.RandomState((case["n"] * 31 + case["nseg"]) % (1 << 31))
        cuts = np.unique(rs.randint(1, case["n"], case["nseg"] - 1))
        off = np.concatenate([[0], cuts, [case["n"]]]).astype(np.int64)
        return off, rs.randint(0, 2, off.size - 1).astype(np.uint8)
    h, S = HIDDEN, case["S"]
    layer = [h * h, KV * h, KV * h, h * h, MLP * h, MLP * h, h * MLP, h, h]
    decay = [1] * 7 + [0, 0]
    if case["segs"] == "model":
        layer = [VOCAB * h] + LAYERS * layer + [VOCAB * h]
        decay = [1] + LAYERS * decay + [1]
    sizes = np.array([max(1, x // S) for x in layer], np.int64)
    return np.concatenate([[0], np.cumsum(sizes)]), np.array(decay, np.uint8)


def _n(case):
    return int(_segments(case)[0][-1])


def _arrays(case):
    """name -> (dtype, count) of the N-sized arrays that the call uses."""
    k, f, b = case["kind"], torch.float32, torch.bfloat16
    a = {}
    if k not in ("reduce_wire",):
        a["master"] = (f, 1)
    if k in ROUNDS or k in ("step", "step_clipped", "reduce_adamw"):
        a["m"] = a["v"] = (f, 1)
    if k not in ("reduce_wire",):
        a["working"] = (b, 1)
    if k not in ("fedavg", "fedopt", "recv"):
        a["grads"] = (b, case["R"] * (1 if case["reuse"] else case["A"]))
    if k in ("round", "round_noalloc", "round_outer", "round_hsdp"):
        a["replicas"] = (b, case["G"] - 1)
    if k in ("fedavg", "fedopt"):
        a["replicas"] = (b, case["G"])
    if k.startswith("round_hsdp"):
        a["wires"] = (b, (case["H"] - 1) * (1 if case["reuse"] else case["A"]))
    if k.startswith("round_hsdp") or k == "reduce_wire":
        a["wire"] = (b, 1)
    if k in ("round_outer", "fedopt"):
        a["prev"] = a["buf"] = (f, 1)
    if k in ("round_hsdp_recv", "recv"):
        a["recv"] = (f, 1)
    if k == "reduce_adamw":
        a["g"] = (f, 1)
    if k in ROUNDS and case["scratch"]:
        a["scratch"] = (f, 1)
    return a


def _state_bytes(case):
    return _n(case) * sum((4 if d is torch.float32 else 2) * c for d, c in _arrays(case).values())


def work(case):
    """Bytes the call cannot do without, each of its passes' inputs read once
    and outputs written once: a local step needs every update of the step
    before, FedAvg the last one, and a clipped step the whole shard's norm
    before its first update (so the gradients twice, or their fp32 sum stored
    and read back, whichever is fewer)."""
    R, G, A, H, n = case["R"], case["G"], case["A"], case["H"], _n(case)
    k = case["kind"]
    hsdp = k.startswith("round_hsdp")
    peers = H if hsdp else R
    step = 2 * peers + 26 + (2 * R + 2 if hsdp else 0)
    if case["clip"] > 0:
        store = case["scratch"] and not hsdp
        step += min(2 * peers, 8) if store else 2 * peers
    fed = 2 * G + 6
    per = {"round": A * step + fed, "round_noalloc": A * step + fed,
           "round_outer": A * step + fed + 16, "round_hsdp": A * step + fed,
           "round_hsdp_recv": A * step + 10, "step": step, "step_clipped": step,
           "reduce_adamw": 2 * R + 4 + 30, "reduce_wire": 2 * R + 2, "fedavg": fed,
           "fedopt": fed + 16, "recv": 10}[k]
    return {"bytes": float(per) * n, "flops": float(n * (A * (R + 20) + 2 * G))}


# ---- inputs ----------------------------------------------------------------


def _fill(case, a, seed, dev="cuda"):
    """Fill the arrays `a` (name -> list of tensors) from the seed."""
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)

    def normal(t, std):
        return t.normal_(0.0, std, generator=gen)

    base = a["master"][0] if "master" in a else None
    if base is not None:
        normal(base, 0.02)
        a["working"][0].copy_(base)
    if "m" in a:
        normal(a["m"][0], 1e-4)
        a["v"][0].uniform_(0.5e-7, 1.5e-7, generator=gen)
    for t in a.get("grads", []):
        normal(t, 1e-3)
        if case["heavy_tails"]:
            # Student-t(3): a normal over the root of a chi-square / 3
            for i in range(0, t.numel(), CHUNK):
                p = t[i:i + CHUNK]
                z = torch.empty((3, p.numel()), device=dev).normal_(generator=gen)
                p.copy_(p.float() / (z.square_().sum(0) / 3).sqrt_())
                p[z[0] < 0.004] = 0      # about one in twenty is exactly zero
    for t in a.get("replicas", []) + a.get("recv", []) + a.get("prev", []):
        normal(t, 1e-4)
        torch.add(t, base, out=t)
    for t in a.get("wires", []):
        normal(t, 1e-3 / case["R"] ** 0.5)
    if "buf" in a:
        normal(a["buf"][0], 1e-4)
    for k in ("wire", "g", "scratch"):
        if k in a:
            a[k][0].zero_()


def _weights(case):
    return [1.0 + (7 * g) % 5 for g in range(case["G"])]


def _lists(case, a):
    """The call's lists: A*R gradients, G replicas, A*H wires."""
    A, R, H = case["A"], case["R"], case["H"]
    g = a.get("grads", [])
    grads = g * A if case["reuse"] else g
    reps = list(a.get("replicas", []))
    if case["kind"] in ROUNDS and case["kind"] != "round_hsdp_recv":
        reps = [None] + reps
    wires = None
    if "wires" in a:
        w = a["wires"]
        wires = []
        for s in range(A):
            mine = w if case["reuse"] else w[s * (H - 1):(s + 1) * (H - 1)]
            wires += [None] + mine
    return grads, reps, wires


def prepare(case, seed):
    n = _n(case)
    plan = _arrays(case)
    flat = iter(P.place_arrays(n, [d for d, c in plan.values() for _ in range(c)], "cuda"))
    a = {k: [next(flat) for _ in range(c)] for k, (d, c) in plan.items()}
    _fill(case, a, seed)
    off, dec = _segments(case)
    s = {k: v[0] for k, v in a.items() if k not in ("grads", "replicas", "wires")}
    s["case"], s["step"] = case, STEP0
    s["layout"] = P.Layout(off, dec)
    s["grads"], s["replicas"], s["wires"] = _lists(case, a)
    s["weights"] = _weights(case)
    rows = case["A"] if case["kind"] in ROUNDS else 1
    s["seg_sumsq"] = (torch.zeros(rows * (off.size - 1), dtype=torch.float32, device="cuda")
                      if case["sumsq"] else None)
    s["total"] = torch.zeros(1, dtype=torch.float64, device="cuda")
    return s


# ---- the pass --------------------------------------------------------------


def run(s):
    c, lay, ss = s["case"], s["layout"], s["seg_sumsq"]
    k, R = c["kind"], c["R"]
    step, s["step"] = s["step"], s["step"] + c["A"]
    out = {}
    if k in ROUNDS:
        cfg = P.make_round_cfg(
            R, c["G"], c["A"], s["weights"], ADAMW, step0=step, max_grad_norm=c["clip"],
            step_lr=_schedule(c, step) if c["clip"] > 0 else None,
            grad_scratch=s.get("scratch"))
        state = (s["master"], s["m"], s["v"], s["working"])
        if k == "round":
            P.fl_round(lay, cfg, s["grads"], s["replicas"], *state, seg_sumsq=ss)
        elif k == "round_noalloc":
            P.fl_round_noalloc(lay, cfg, s["grads"], s["replicas"], *state, seg_sumsq=ss)
        elif k == "round_outer":
            P.fl_round_outer(lay, cfg, OUTER, s["grads"], s["replicas"], s["prev"], s["buf"],
                             *state, seg_sumsq=ss)
        else:
            member = k == "round_hsdp"
            hc = P.make_hsdp_cfg(c["H"], 0, None, member)
            P.fl_round_hsdp(lay, cfg, hc, s["grads"], s["wires"], s["wire"],
                            s["replicas"] if member else None,
                            None if member else s["recv"], *state, seg_sumsq=ss)
    elif k == "step":
        P.fl_local_step(lay, ADAMW, step, s["grads"], 1.0 / R, s["master"], s["m"], s["v"],
                        s["working"], seg_sumsq=ss)
    elif k == "step_clipped":
        P.fl_grad_sumsq(lay, s["grads"], 1.0 / R, s["total"], seg_sumsq=ss)
        P.fl_local_step_clipped(lay, ADAMW, step, s["grads"], 1.0 / R, s["total"], c["clip"],
                                s["master"], s["m"], s["v"], s["working"])
        out["total"] = s["total"]
    elif k == "reduce_adamw":
        P.fl_shard_reduce(lay, s["grads"], 1.0 / R, s["g"], seg_sumsq=ss)
        P.fl_adamw_step(lay, ADAMW, step, s["g"], s["master"], s["m"], s["v"], s["working"])
        out["g"] = s["g"]
    elif k == "reduce_wire":
        P.fl_shard_reduce_wire(lay, s["grads"], 1.0 / R, s["wire"])
        return {"wire": s["wire"]}
    elif k == "fedavg":
        P.fl_fedavg(lay, s["replicas"], s["weights"], s["master"], s["working"])
    elif k == "fedopt":
        P.fl_fedopt(lay, s["replicas"], s["weights"], OUTER, s["prev"], s["buf"], s["master"],
                    s["working"])
    else:
        P.fl_broadcast_recv(lay, s["recv"], s["master"], s["working"])
    for x in ("master", "m", "v", "working", "wire", "prev", "buf"):
        if x in s:
            out[x] = s[x]
    if ss is not None:
        out["seg_sumsq"] = ss
    return out


def _schedule(case, step):
    total, warm = SCHEDULE
    return [P.lr_cosine(step + a, total, warm, ADAMW["lr"]) for a in range(case["A"])]


# ---- the same in 64 bits -----------------------------------------------------


def tolerance(case):
    """Sums and moments are within 1.3e-7 of their 64-bit values.  What is
    wider is the bf16 rounding of a working copy or wire shard whose fp32
    value moved across a tie: rare, one bf16 step (2^-7 of the value), and
    carried into the average (up to 7e-6 of it), and into the outer momentum
    (8e-5), which is the small difference of two models.  Four times that."""
    if case["kind"] in ("round_outer", "fedopt"):
        return {"rel": 3e-4, "max": 0.3}
    return {"rel": 3e-5, "max": 0.01}


def _f32(x):
    return float(np.float32(x))


def _exact_lr(case, step):
    if case["clip"] <= 0 or case["kind"] not in ROUNDS:
        return ADAMW["lr"]
    total, warm = SCHEDULE
    s = step - 1
    f = s / warm if s < warm else 0.5 * (1 + np.cos(np.pi * (s - warm) / (total - warm)))
    return ADAMW["lr"] * f


def exact(case, seed):
    n, k = _n(case), case["kind"]
    plan = _arrays(case)
    a = {x: [torch.empty(n, dtype=d, device="cuda") for _ in range(c)]
         for x, (d, c) in plan.items()}
    _fill(case, a, seed)
    grads, reps, wires = _lists(case, a)
    off, dec = _segments(case)
    n_seg = off.size - 1
    R, A, H = case["R"], case["A"], case["H"]
    hsdp = k.startswith("round_hsdp")
    steps = A if k in ROUNDS else (1 if k in ("step", "step_clipped", "reduce_adamw") else 0)
    d64 = torch.float64
    spans = [(i, min(n, i + CHUNK)) for i in range(0, n, CHUNK)]
    out = {}

    def mean(ts, i, j, scale):
        acc = torch.zeros(j - i, dtype=d64, device="cuda")
        for t in ts:
            acc += t[i:j].double()
        return acc * scale

    def bf16(x):
        return x.float().bfloat16()

    def gradient(s, i, j):
        """The averaged gradient that step s applies, and the wire shard."""
        g = mean(grads[s * R:(s + 1) * R], i, j, 1.0 / R)
        if not hsdp:
            return g, None
        w = bf16(g)
        return (w.double() + mean(wires[s * H + 1:(s + 1) * H], i, j, 1.0)) / H, w

    if k == "reduce_wire":
        wire = torch.empty(n, dtype=d64, device="cuda")
        for i, j in spans:
            wire[i:j] = mean(grads, i, j, 1.0 / R)
        return {"wire": wire}

    # per-segment sums of squares of each step's gradient (float64 sums of
    # the segments' parts in each span)
    sums = np.zeros((max(steps, 1), n_seg))
    if case["sumsq"] or case["clip"] > 0:
        seen = {}
        for s in range(steps):
            key = tuple(t.data_ptr() for t in grads[s * R:(s + 1) * R])
            if key in seen:
                sums[s] = sums[seen[key]]
                continue
            seen[key] = s
            for i, j in spans:
                sq = gradient(s, i, j)[0].square_()
                lo = int(np.searchsorted(off, i, side="right")) - 1
                hi = int(np.searchsorted(off, j, side="left"))
                edges = np.clip(off[lo:hi + 1], i, j) - i
                lens = torch.from_numpy(np.diff(edges)).cuda()
                sums[s, lo:hi] += torch.segment_reduce(sq, "sum", lengths=lens).cpu().numpy()
    names = [x for x in ("master", "m", "v", "working", "wire", "prev", "buf", "g") if x in plan]
    for x in names:
        out[x] = torch.empty(n, dtype=d64, device="cuda")
    dec_t = torch.from_numpy(dec.astype(np.float64)).cuda()
    off_t = torch.from_numpy(off[1:]).cuda()
    h = {x: _f32(y) for x, y in ADAMW.items()}
    w = np.array(_weights(case)) / sum(_weights(case))
    for i, j in spans:
        p = a["master"][0][i:j].double()
        work_copy = a["working"][0][i:j]
        if steps:
            m, v = a["m"][0][i:j].double(), a["v"][0][i:j].double()
            flag = dec_t[torch.searchsorted(off_t, torch.arange(i, j, device="cuda"), right=True)]
        for s in range(steps):
            g, wire = gradient(s, i, j)
            if wire is not None:
                out["wire"][i:j] = wire
            if "g" in out:
                out["g"][i:j] = g
            if case["clip"] > 0:
                norm = np.sqrt(sums[s].sum())
                g = g * min(1.0, _f32(case["clip"]) / (norm + 1e-6))
            t, lr = STEP0 + s, _f32(_exact_lr(case, STEP0 + s))
            p = p * (1 - lr * h["weight_decay"] * flag)
            m = h["beta1"] * m + (1 - h["beta1"]) * g
            v = h["beta2"] * v + (1 - h["beta2"]) * g * g
            den = (v / (1 - h["beta2"] ** t)).sqrt() + h["eps"]
            p = p - lr / (1 - h["beta1"] ** t) * m / den
            work_copy = bf16(p)
        if k in ("recv", "round_hsdp_recv"):
            p = a["recv"][0][i:j].double()
        elif k in ROUNDS or k in ("fedavg", "fedopt"):
            avg = torch.zeros_like(p)
            for g, r in enumerate(reps):
                avg += w[g] * (work_copy if r is None else r[i:j]).double()
            p = avg
        if k in ("round_outer", "fedopt"):
            prev, buf = a["prev"][0][i:j].double(), a["buf"][0][i:j].double()
            delta = prev - avg
            buf = _f32(OUTER["momentum"]) * buf + delta
            p = prev - _f32(OUTER["lr"]) * (delta + _f32(OUTER["momentum"]) * buf)
            out["prev"][i:j], out["buf"][i:j] = p, buf
        out["master"][i:j] = p
        out["working"][i:j] = p
        if steps:
            out["m"][i:j], out["v"][i:j] = m, v
    if k == "step_clipped":
        out["total"] = torch.tensor([sums[0].sum()], dtype=d64)
    if case["sumsq"]:
        out["seg_sumsq"] = torch.from_numpy(sums.reshape(-1))
    return out
