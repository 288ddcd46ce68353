"""The order in which the sums of squares are added.

It is one fixed tree over element indices, whatever kernel, launch shape or
exchange computes it: a lane's 8 consecutive squares in order, a butterfly
over the 64 lanes of a unit of 512 elements (lanes 32, 16, 8, 4, 2 and 1
apart), the four units of each (tile of 2048, segment) piece in the
finalize's trees.  The tree is written out here in numpy, double for double.

The gradients are such that the order decides the result's bits: a segment
holds one 1 and one 2^-12 among some 2^-27, so that its sum of squares is half
a float step past 1, and a square of 2^-54 is lost when it meets the 1 on its
own and counts when it comes with others.  The float rounding of the sum is 1
or 1 + 2^-23 accordingly.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

ADAMW = dict(lr=3e-4, beta1=0.9, beta2=0.95, eps=1e-8, weight_decay=0.1)
TILE, UNIT, CHUNK = 2048, 512, 1024


@pytest.fixture(scope="module")
def env():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_20359_amd as P

    P.lib()
    return torch, P


# ---- the tree ----------------------------------------------------------------


def butterfly(v):
    """Sum of 64 lanes; v: (..., 64) doubles."""
    lane = np.arange(64)
    for off in (32, 16, 8, 4, 2, 1):
        v = v + v[..., lane ^ off]
    return v[..., 0]


def fold256(v):
    """Thread j of 256 adds v[j], v[j + 256], ... (rows in order), then the
    four waves' butterflies in order; v: (k, w) doubles, w added in order."""
    acc = np.zeros(256)
    for k in range(0, v.shape[0], 256):
        part = v[k:k + 256]
        for w in range(v.shape[1]):
            acc[:part.shape[0]] = acc[:part.shape[0]] + part[:, w]
    r = butterfly(acc.reshape(4, 64))
    return ((r[0] + r[1]) + r[2]) + r[3]


def segment_sum(x, lo, hi):
    """Sum of squares of the float32 segment x = elements lo .. hi - 1."""
    t0, t1 = lo // TILE, (hi - 1) // TILE + 1
    sq = np.zeros((t1 - t0) * TILE)
    sq[lo - t0 * TILE:hi - t0 * TILE] = x.astype(np.float64) ** 2
    lanes = sq.reshape(-1, 64, 8)
    acc = np.zeros(lanes.shape[:2])
    for e in range(8):
        acc = acc + lanes[..., e]
    pieces = butterfly(acc).reshape(-1, TILE // UNIT)
    total = 0.0
    for c in range(0, pieces.shape[0], CHUNK):
        total = total + fold256(pieces[c:c + CHUNK])
    return total


# ---- gradients whose order shows -----------------------------------------------


def shaped(lengths, seed):
    """Segment offsets and a float32 gradient (bf16 values)."""
    r = np.random.default_rng(seed)
    off = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    g = np.zeros(off[-1], np.float32)
    for lo, hi in zip(off[:-1], off[1:]):
        k = r.integers(3, 7)
        at = lo + r.permutation(min(hi - lo, 700))[:k + 2]
        g[at[2:]] = 2.0 ** -27
        g[at[0]], g[at[1]] = 1.0, 2.0 ** -12
    return off, g


def lengths(seed):
    """Whole units, odd cuts through units and tiles, a tail cut short."""
    r = np.random.default_rng(seed)
    return np.concatenate([[512] * 8, r.integers(40, 600, 40), [2048, 4096 + 7], [301]])


def expected(off, g):
    segs = [segment_sum(g[lo:hi], lo, hi) for lo, hi in zip(off[:-1], off[1:])]
    return np.array(segs), fold256(np.array(segs)[:, None])


def on_device(torch, g):
    return torch.from_numpy(g).cuda().bfloat16()


def test_shaped_gradients_show_the_order():
    """On the CPU: other orders give other floats for many of the segments."""
    off, g = shaped(lengths(1), 1)
    segs, _ = expected(off, g)
    up = np.float32(segs) > 1
    assert 10 < up.sum() < up.size - 10
    plain = np.array([np.cumsum(g[lo:hi].astype(np.float64) ** 2)[-1]
                      for lo, hi in zip(off[:-1], off[1:])])
    assert (np.float32(plain) != np.float32(segs)).sum() > 5


def long_layout(torch, P, off, g):
    """The shaped segments at both ends of a shard of 384 units per CU, where
    long passes begin, zeros between; (layout, gradient, shaped sums)."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    n0 = int(off[-1])
    mid = 384 * cus * UNIT
    at = n0 + mid
    full = np.concatenate([off, at + off])
    t = torch.zeros(at + n0, dtype=torch.bfloat16, device="cuda")
    t[:n0] = on_device(torch, g)
    t[at:] = t[:n0]
    ends = np.array([segment_sum(g[a:b], at + a, at + b) for a, b in zip(off[:-1], off[1:])])
    head = [segment_sum(g[a:b], a, b) for a, b in zip(off[:-1], off[1:])]
    return P.Layout(full, np.ones(full.size - 1, np.uint8)), t, np.concatenate([head, [0.0], ends])


def peers_of(torch, t, R):
    """R streams whose sum is t: t last, zeros before it."""
    return [torch.zeros_like(t)] * (R - 1) + [t]


def state(torch, n):
    p, m = torch.zeros(n, device="cuda"), torch.zeros(n, device="cuda")
    return p, m, torch.full((n,), 1e-7, device="cuda"), torch.zeros(n, dtype=torch.bfloat16,
                                                                    device="cuda")


@pytest.mark.parametrize("R", [1, 2, 3, 8, 9, 26])
def test_total_is_the_tree(env, R):
    """The whole-shard total as a double, and the segments' floats."""
    torch, P = env
    off, g = shaped(lengths(R), R)
    segs, total = expected(off, g)
    lay = P.Layout(off, np.ones(off.size - 1, np.uint8))
    got = torch.zeros(1, dtype=torch.float64, device="cuda")
    ss = torch.zeros(off.size - 1, device="cuda")
    print("total R=%d n=%d" % (R, g.size), flush=True)
    P.fl_grad_sumsq(lay, peers_of(torch, on_device(torch, g), R), 1.0, got, seg_sumsq=ss)
    assert float(got) == total
    assert np.array_equal(ss.cpu().numpy(), np.float32(segs))
    lay.close()


@pytest.mark.parametrize("R", [3, 12])
def test_long_and_short_steps_agree(env, R):
    """The step's two exchanges (by lanes on a short shard, by way of LDS on a
    long one) give a segment the same float."""
    torch, P = env
    off, g = shaped(lengths(R), R)
    n0 = int(off[-1])
    short = P.Layout(off, np.ones(off.size - 1, np.uint8))
    ss = torch.zeros(off.size - 1, device="cuda")
    print("step R=%d short" % R, flush=True)
    P.fl_local_step(short, ADAMW, 9, peers_of(torch, on_device(torch, g), R), 1.0,
                    *state(torch, n0), seg_sumsq=ss)
    lay, t, want = long_layout(torch, P, off, g)
    long_ss = torch.zeros(2 * (off.size - 1) + 1, device="cuda")
    print("step R=%d long n=%d" % (R, t.numel()), flush=True)
    P.fl_local_step(lay, ADAMW, 9, peers_of(torch, t, R), 1.0, *state(torch, t.numel()),
                    seg_sumsq=long_ss)
    assert torch.equal(long_ss[:off.size - 1], ss)
    assert np.array_equal(ss.cpu().numpy(), np.float32(expected(off, g)[0]))
    assert np.array_equal(long_ss.cpu().numpy(), np.float32(want))
    short.close()
    lay.close()


@pytest.mark.parametrize("R", [1, 2, 3, 8, 9, 26])
def test_every_pass_adds_in_one_order(env, R):
    """The reduction to fp32, the sums alone and the fused step, whose lanes
    hold different elements, and a clipped round with and without the gradient
    scratch: the same segments' floats, and the same state."""
    torch, P = env
    off, g = shaped(lengths(20 + R), 20 + R)
    n = int(off[-1])
    want = np.float32(expected(off, g)[0])
    lay = P.Layout(off, np.ones(off.size - 1, np.uint8))
    peers = peers_of(torch, on_device(torch, g), R)
    ss = torch.zeros(off.size - 1, device="cuda")
    print("passes R=%d n=%d" % (R, n), flush=True)
    P.fl_shard_reduce(lay, peers, 1.0, torch.empty(n, device="cuda"), seg_sumsq=ss)
    assert np.array_equal(ss.cpu().numpy(), want)
    P.fl_grad_sumsq(lay, peers, 1.0, torch.zeros(1, dtype=torch.float64, device="cuda"),
                    seg_sumsq=ss.zero_())
    assert np.array_equal(ss.cpu().numpy(), want)
    P.fl_local_step(lay, ADAMW, 9, peers, 1.0, *state(torch, n), seg_sumsq=ss.zero_())
    assert np.array_equal(ss.cpu().numpy(), want)
    out = []
    for scratch in (None, torch.empty(n, device="cuda")):
        cfg = P.make_round_cfg(R, 1, 1, [1.0], ADAMW, step0=9, grad_scale=1.0, max_grad_norm=1.0,
                               grad_scratch=scratch)
        st = state(torch, n)
        P.fl_round(lay, cfg, peers, [None], *st, seg_sumsq=ss.zero_())
        assert np.array_equal(ss.cpu().numpy(), want)
        out.append(st)
    assert all(torch.equal(a, b) for a, b in zip(*out))
    lay.close()
