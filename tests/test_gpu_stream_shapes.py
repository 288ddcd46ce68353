"""The streaming passes at the edges of their shapes: every number of streams
around the compile-time counts and the chunks of the generic one, units (512
elements) and tiles cut short, and shard lengths around the bands in which the
launch shape changes; against the oracle, bit for bit."""
import numpy as np
import pytest

import harness as H

pytestmark = pytest.mark.gpu

ADAMW = dict(lr=3e-4, beta1=0.9, beta2=0.95, eps=1e-8, weight_decay=0.1)


@pytest.fixture(scope="module")
def env():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import oracle
    import paper_2609_20359_amd as P

    P.lib()
    return torch, P, oracle.Oracle()


def _bf16(torch, n, std, k):
    g = torch.Generator(device="cuda")
    g.manual_seed(1000 + k)
    return torch.empty(n, dtype=torch.bfloat16, device="cuda").normal_(0.0, std, generator=g)


def _layout(P, n, n_seg, seed):
    r = np.random.default_rng(seed)
    cuts = np.unique(r.integers(1, n, n_seg - 1)) if n_seg > 1 and n > 1 else []
    off = np.concatenate([[0], cuts, [n]]).astype(np.int64)
    dec = r.integers(0, 2, off.size - 1).astype(np.uint8)
    return off, dec, P.Layout(off, dec)


@pytest.mark.parametrize("K", [1, 2, 3, 4, 5, 6, 7, 8, 9, 15, 16, 17, 23, 24, 31, 64])
@pytest.mark.parametrize("n", [511, 513, 4 * 512 + 1, 20_483])
def test_stream_counts(env, K, n):
    torch, P, orc = env
    off, dec, lay = _layout(P, n, 9, n + K)
    peers = [_bf16(torch, n, 1e-3, k) for k in range(K)]
    host = [H.to_u16(t) for t in peers]
    scale = 1.0 / K
    print("streams K=%d n=%d" % (K, n), flush=True)

    g = torch.empty(n, device="cuda")
    ss = torch.full((off.size - 1,), -1.0, device="cuda")
    P.fl_shard_reduce(lay, peers, scale, g, seg_sumsq=ss)
    want = orc.shard_reduce(host, scale)
    assert np.array_equal(g.cpu().numpy().view(np.uint32), want.view(np.uint32))
    ref = orc.seg_sumsq(off, want)
    H.assert_sumsq("reduce", ss.cpu().numpy(), ref)
    total = torch.zeros(1, dtype=torch.float64, device="cuda")
    only = torch.full_like(ss, -1.0)
    P.fl_grad_sumsq(lay, peers, scale, total, seg_sumsq=only)
    assert torch.equal(only, ss)
    assert abs(float(total) - ref.sum()) <= 1e-12 * ref.sum()
    wire = torch.empty(n, dtype=torch.bfloat16, device="cuda")
    P.fl_shard_reduce_wire(lay, peers, scale, wire)
    assert np.array_equal(H.to_u16(wire), orc.shard_reduce_wire(host, scale))

    master = torch.empty(n, device="cuda").normal_(0.0, 0.02)
    m, v = torch.empty(n, device="cuda").normal_(0.0, 1e-4), torch.full((n,), 1e-7, device="cuda")
    work = torch.empty(n, dtype=torch.bfloat16, device="cuda")
    rm, r1, r2 = (t.cpu().numpy().copy() for t in (master, m, v))
    rw = np.zeros(n, np.uint16)
    step = torch.full_like(ss, -1.0)
    P.fl_local_step(lay, ADAMW, 7, peers, scale, master, m, v, work, seg_sumsq=step)
    orc.adamw_step(off, dec, ADAMW, 7, want, rm, r1, r2, rw)
    H.assert_state_parity("step", dict(master=master.cpu().numpy(), m=m.cpu().numpy(),
                                       v=v.cpu().numpy(), working=H.to_u16(work)),
                          dict(master=rm, m=r1, v=r2, working=rw), bitwise=True)
    assert torch.equal(step, ss)

    weights = 1.0 + np.arange(K) % 5
    P.fl_fedavg(lay, peers, weights, master, work)
    rm, rw = orc.fedavg(host, weights)
    assert np.array_equal(master.cpu().numpy().view(np.uint32), rm.view(np.uint32))
    assert np.array_equal(H.to_u16(work), rw)
    lay.close()


# The last unit when the shard's end cuts it: in either half, at and inside a
# group of four, and shards of less than a group.
@pytest.mark.parametrize("K", [1, 4, 5, 8, 9, 64])
@pytest.mark.parametrize("n", [1, 2, 3, 5, 8, 254, 256, 257, 259, 510, 512 + 4, 4 * 512 - 1])
def test_cut_units(env, K, n):
    torch, P, orc = env
    test_stream_counts(env, K, n)
    off, dec, lay = _layout(P, n, 3, n + K)
    reps = [_bf16(torch, n, 2e-2, k) for k in range(K)]
    weights = 1.0 + np.arange(K) % 3
    outer = dict(lr=0.7, momentum=0.9, nesterov=False)
    prev, buf = (torch.empty(n, device="cuda").normal_(0.0, s) for s in (0.02, 1e-4))
    master, recv = torch.empty(n, device="cuda"), torch.empty(n, device="cuda").normal_()
    work = torch.empty(n, dtype=torch.bfloat16, device="cuda")
    rp, rb, rm = (t.cpu().numpy().copy() for t in (prev, buf, master))
    rw = np.zeros(n, np.uint16)
    print("cut outer K=%d n=%d" % (K, n), flush=True)
    P.fl_fedopt(lay, reps, weights, outer, prev, buf, master, work)
    orc.fedopt([H.to_u16(t) for t in reps], weights, outer, rp, rb, rm, rw)
    for t, r in ((prev, rp), (buf, rb), (master, rm)):
        assert np.array_equal(t.cpu().numpy().view(np.uint32), r.view(np.uint32))
    assert np.array_equal(H.to_u16(work), rw)
    P.fl_broadcast_recv(lay, recv, master, work)
    assert torch.equal(master, recv) and torch.equal(work, recv.bfloat16())
    lay.close()


# Units of several segments: tiles of up to 64 (a lane for each) and of more
# (search); at a mean of 32 elements tiles have a few less and a few more than 64.
@pytest.mark.parametrize("R", [1, 4, 9, 26])
@pytest.mark.parametrize("mean", [1, 3, 32, 37, 700])
def test_short_segments(env, R, mean):
    torch, P, orc = env
    n = 11 * 2048 + 515
    r = np.random.default_rng(mean)
    cuts = np.unique(r.integers(1, n, n // mean)) if mean > 1 else np.arange(1, n)
    off = np.concatenate([[0], cuts, [n]]).astype(np.int64)
    dec = r.integers(0, 2, off.size - 1).astype(np.uint8)
    if mean == 32:
        per = [np.sum((off[:-1] < t + 2048) & (off[1:] > t)) for t in range(0, n, 2048)]
        assert min(per[:-1]) <= 64 < max(per)
    lay = P.Layout(off, dec)
    peers = [_bf16(torch, n, 1e-3, k) for k in range(R)]
    want = orc.shard_reduce([H.to_u16(t) for t in peers], 1.0 / R)
    ref = orc.seg_sumsq(off, want)
    p0, m0 = torch.empty(n, device="cuda").normal_(0.0, 0.02), torch.full((n,), 1e-5, device="cuda")
    rm, r1, r2, rw = p0.cpu().numpy(), m0.cpu().numpy(), m0.cpu().numpy() ** 2, np.zeros(n, np.uint16)
    orc.adamw_step(off, dec, ADAMW, 7, want, rm, r1, r2, rw)
    for ss in (None, torch.full((off.size - 1,), -1.0, device="cuda")):
        master, m = p0.clone(), m0.clone()
        v, work = m0 ** 2, torch.empty(n, dtype=torch.bfloat16, device="cuda")
        print("segments of %d R=%d sums=%s" % (mean, R, ss is not None), flush=True)
        P.fl_local_step(lay, ADAMW, 7, peers, 1.0 / R, master, m, v, work, seg_sumsq=ss)
        H.assert_state_parity("step", dict(master=master.cpu().numpy(), m=m.cpu().numpy(),
                                           v=v.cpu().numpy(), working=H.to_u16(work)),
                              dict(master=rm, m=r1, v=r2, working=rw.copy()), bitwise=True)
    H.assert_sumsq("step", ss.cpu().numpy(), ref)
    total = torch.zeros(1, dtype=torch.float64, device="cuda")
    P.fl_grad_sumsq(lay, peers, 1.0 / R, total, seg_sumsq=ss.fill_(-1.0))
    H.assert_sumsq("sums", ss.cpu().numpy(), ref)
    P.fl_shard_reduce(lay, peers, 1.0 / R, m, seg_sumsq=ss.fill_(-1.0))
    H.assert_sumsq("reduce", ss.cpu().numpy(), ref)
    lay.close()


def test_cut_units_write_nothing_past_the_end(env):
    """What lies behind a shard's arrays stays as it is."""
    torch, P, _ = env
    room = 512
    for n in (1, 3, 255, 257, 513, 1022):
        off, dec, lay = _layout(P, n, 1, n)

        def arr(dt, fill):
            return torch.full((n + room,), fill, dtype=dt, device="cuda")

        g = [arr(torch.bfloat16, 1e-3) for _ in range(3)]
        f = {k: arr(torch.float32, 0.25) for k in ("g", "master", "m", "v", "prev", "buf")}
        w = arr(torch.bfloat16, 0.25)
        s = {k: t[:n] for k, t in f.items()}
        gs = [t[:n] for t in g]
        print("past the end n=%d" % n, flush=True)
        P.fl_shard_reduce(lay, gs, 1.0, s["g"])
        P.fl_shard_reduce_wire(lay, gs, 1.0, w[:n])
        P.fl_local_step(lay, ADAMW, 1, gs, 1.0, s["master"], s["m"], s["v"], w[:n])
        P.fl_adamw_step(lay, ADAMW, 1, s["g"], s["master"], s["m"], s["v"], w[:n])
        P.fl_fedavg(lay, gs, [1.0] * 3, s["master"], w[:n])
        P.fl_fedopt(lay, gs, [1.0] * 3, dict(lr=0.7, momentum=0.9, nesterov=True), s["prev"],
                    s["buf"], s["master"], w[:n])
        P.fl_broadcast_recv(lay, s["v"], s["master"], w[:n])
        for t in list(f.values()) + [w]:
            assert torch.equal(t[n:], torch.full_like(t[n:], 0.25))
        lay.close()


def test_cut_unit_costs_no_more_than_a_whole_one(env):
    """64 streams: a shard of one unit less an element, and the whole unit (one
    element and stream after another, the first took 70 us, the second 33, which
    is the call from Python)."""
    torch, P, _ = env

    def us(n, reps=40):
        _, _, lay = _layout(P, n, 1, n)
        peers = [_bf16(torch, n, 1e-3, k) for k in range(64)]
        wire = torch.empty(n, dtype=torch.bfloat16, device="cuda")
        best = float("inf")
        for _ in range(8):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            for _ in range(reps):
                P.fl_shard_reduce_wire(lay, peers, 1.0, wire)
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b) * 1e3 / reps)
        lay.close()
        return best

    whole, cut = us(512), us(511)
    print("one unit %.1f us, less an element %.1f us" % (whole, cut), flush=True)
    assert cut < 1.5 * whole


# Units per CU on both sides of each threshold of the launch shape (no limit up
# to 20; from 100 and from 384 on), at whole and at ragged lengths.
@pytest.mark.parametrize("units,more", [(20, 0), (21, 3), (99, 3), (100, 0), (383, 3), (384, 0),
                                        (384, 3)])
def test_launch_bands(env, units, more):
    torch, P, orc = env
    n = units * 512 * torch.cuda.get_device_properties(0).multi_processor_count + more
    off, dec, lay = _layout(P, n, 40, n)
    for K in (1, 2, 3):
        print("band n=%d K=%d" % (n, K), flush=True)
        peers = [_bf16(torch, n, 1e-3, k) for k in range(K)]
        host = [H.to_u16(t) for t in peers]
        want = orc.shard_reduce(host, 1.0 / K)
        total = torch.zeros(1, dtype=torch.float64, device="cuda")
        ss = torch.full((off.size - 1,), -1.0, device="cuda")
        P.fl_grad_sumsq(lay, peers, 1.0 / K, total, seg_sumsq=ss)
        H.assert_sumsq("sumsq", ss.cpu().numpy(), orc.seg_sumsq(off, want))
        g = torch.empty(n, device="cuda")
        P.fl_shard_reduce(lay, peers, 1.0 / K, g)
        assert np.array_equal(g.cpu().numpy().view(np.uint32), want.view(np.uint32))
        wire = torch.empty(n, dtype=torch.bfloat16, device="cuda")
        P.fl_shard_reduce_wire(lay, peers, 1.0 / K, wire)
        assert np.array_equal(H.to_u16(wire), orc.shard_reduce_wire(host, 1.0 / K))
    master = torch.empty(n, device="cuda").normal_(0.0, 0.02)
    m, v = torch.empty(n, device="cuda").normal_(0.0, 1e-4), torch.full((n,), 1e-7, device="cuda")
    work = torch.empty(n, dtype=torch.bfloat16, device="cuda")
    rm, r1, r2 = (t.cpu().numpy().copy() for t in (master, m, v))
    rw = np.zeros(n, np.uint16)
    ss.fill_(-1.0)   # (units cut by segment boundaries, at three peers)
    P.fl_local_step(lay, ADAMW, 3, peers, 1.0 / 3, master, m, v, work, seg_sumsq=ss)
    orc.adamw_step(off, dec, ADAMW, 3, want, rm, r1, r2, rw)
    H.assert_state_parity("step", dict(master=master.cpu().numpy(), m=m.cpu().numpy(),
                                       v=v.cpu().numpy(), working=H.to_u16(work)),
                          dict(master=rm, m=r1, v=r2, working=rw), bitwise=True)
    H.assert_sumsq("step", ss.cpu().numpy(), orc.seg_sumsq(off, want))

    print("band n=%d FedAvg, outer step, receive" % n, flush=True)
    weights = [1.0, 2.0, 3.0]
    P.fl_fedavg(lay, peers, weights, master, work)
    fm, fw = orc.fedavg(host, weights)
    assert np.array_equal(master.cpu().numpy().view(np.uint32), fm.view(np.uint32))
    assert np.array_equal(H.to_u16(work), fw)
    outer = dict(lr=0.7, momentum=0.9, nesterov=True)
    prev, buf = (torch.empty(n, device="cuda").normal_(0.0, s) for s in (0.02, 1e-4))
    rp, rb = prev.cpu().numpy().copy(), buf.cpu().numpy().copy()
    P.fl_fedopt(lay, peers, weights, outer, prev, buf, master, work)
    orc.fedopt(host, weights, outer, rp, rb, rm, rw)
    for t, r in ((prev, rp), (buf, rb), (master, rm)):
        assert np.array_equal(t.cpu().numpy().view(np.uint32), r.view(np.uint32))
    assert np.array_equal(H.to_u16(work), rw)
    P.fl_broadcast_recv(lay, m, prev, work)
    assert torch.equal(prev, m) and torch.equal(work, m.bfloat16())
    lay.close()


@pytest.mark.parametrize("eps,beta2", [(1e-8, 0.95), (1e-30, 0.999), (1e15, 0.9999999),
                                       (2.0 ** -60, 0.0)])
@pytest.mark.parametrize("t", [1, 1000])
def test_adamw_operand_ranges(env, eps, beta2, t):
    """Moments inside, across and beyond the range of the short forms of the
    root and the divisions, whole waves and single lanes of them."""
    torch, P, orc = env
    n = 512 * 24 + 77
    r = np.random.default_rng(int(t * 1000 + beta2 * 100))
    off = np.array([0, n], np.int64)
    dec = np.ones(1, np.uint8)
    unit = np.arange(n) // 512

    def spread(lo, hi):
        x = np.ldexp(r.uniform(1.0, 2.0, n), r.integers(lo, hi, n)) * r.choice([-1.0, 1.0], n)
        return x.astype(np.float32)

    g, m, v = spread(-14, -6), spread(-14, -6), np.abs(spread(-30, -14))
    wide = unit % 3 == 1                       # any magnitude, subnormals among them
    g[wide], m[wide] = spread(-149, 60)[wide], spread(-149, 60)[wide]
    v[wide] = np.abs(spread(-149, 100))[wide]
    one = (unit % 3 == 2) & (r.random(n) < 0.003)   # single lanes
    for a, x in ((g, 0.0), (m, 0.0), (v, 0.0)):
        a[one] = x
    edge = (unit % 6 == 5) & (r.random(n) < 0.003)
    m[edge] = np.float32(2.0 ** -60) * r.choice([0.5, 1.0, 2.0], edge.sum()).astype(np.float32)
    v[edge] = np.float32(2.0 ** -100) * r.choice([0.5, 1.0, 2.0], edge.sum()).astype(np.float32)
    g[edge] = 0.0
    p = spread(-10, -2)
    hp = dict(lr=3e-4, beta1=0.9, beta2=beta2, eps=eps, weight_decay=0.1)
    lay = P.Layout(off, dec)
    dev = [torch.from_numpy(x.copy()).cuda() for x in (g, p, m, v)]
    work = torch.empty(n, dtype=torch.bfloat16, device="cuda")
    print("adamw ranges eps=%g beta2=%g t=%d" % (eps, beta2, t), flush=True)
    P.fl_adamw_step(lay, hp, t, dev[0], dev[1], dev[2], dev[3], work)
    rw = np.zeros(n, np.uint16)
    orc.adamw_step(off, dec, hp, t, g, p, m, v, rw)
    H.assert_state_parity("ranges", dict(master=dev[1].cpu().numpy(), m=dev[2].cpu().numpy(),
                                         v=dev[3].cpu().numpy(), working=H.to_u16(work)),
                          dict(master=p, m=m, v=v, working=rw), bitwise=True)
    lay.close()


def test_every_float_to_bf16(env):
    """The conversion of all 2^32 floats, by the broadcast receive, against
    rounding to nearest even on the bits (a NaN keeps its sign and upper bits
    and becomes quiet)."""
    torch, P, _ = env
    n = 1 << 28
    lay = P.Layout(np.array([0, n], np.int64), np.ones(1, np.uint8))
    master = torch.empty(n, device="cuda")
    work = torch.empty(n, dtype=torch.bfloat16, device="cuda")
    for k in range(16):
        print("floats %d of 16" % k, flush=True)
        lo = (k << 28) - (1 << 31)
        bits = torch.arange(lo, lo + n, dtype=torch.int64, device="cuda")
        recv = bits.to(torch.int32).view(torch.float32)
        P.fl_broadcast_recv(lay, recv, master, work)
        assert torch.equal(master.view(torch.int32), recv.view(torch.int32))
        bits &= 0xFFFFFFFF
        want = (bits + 0x7FFF + ((bits >> 16) & 1)) >> 16
        want = torch.where((bits & 0x7FFFFFFF) > 0x7F800000, (bits >> 16) | 0x40, want)
        got = work.view(torch.int16).to(torch.int64) & 0xFFFF
        assert torch.equal(got, want)
    lay.close()


@pytest.mark.parametrize("exponent,t", [(-100, 1000), (0, 1000), (58, 1000), (0, 1)])
def test_every_mantissa_of_the_root(env, exponent, t):
    """The short form of the root for all floats of two binades: at both ends
    of its range and in the middle, the bias correction 1 (t = 1000) or the
    root of a half.  With these hyperparameters a step halves m and v and moves
    p from 0 to -lr_t m / (sqrt(v) / bc2 + eps), and with m just under the
    denominator the quotient shows each unit in the last place of the root."""
    torch, P, _ = env
    hp = dict(lr=1.0, beta1=0.5, beta2=0.5, eps=2.0 ** -60, weight_decay=0.0)
    f = np.float32
    one = (np.arange(1 << 23, dtype=np.uint32) | np.uint32(127 << 23)).view(f)
    v = np.concatenate([np.ldexp(one, exponent), np.ldexp(one, exponent + 1)])
    bc2, lr = f(np.sqrt(1.0 - 0.5 ** t)), f(1.0 / (1.0 - 0.5 ** t))

    def quotient(root, m):
        return m / (root / bc2 + f(2.0 ** -60))

    root = np.sqrt(v)
    m = (root / bc2 + f(2.0 ** -60)) * f(1.0 - 2.0 ** -21)
    want = quotient(root, m)
    assert m.dtype == want.dtype == f
    if t == 1000:   # (an error in the root shows)
        for to in (np.inf, 0.0):
            assert np.mean(quotient(np.nextafter(root, f(to)), m) == want) < 1e-3
    lay = P.Layout(np.array([0, v.size], np.int64), np.ones(1, np.uint8))
    g, p = torch.zeros(v.size, device="cuda"), torch.zeros(v.size, device="cuda")
    dm, dv = torch.from_numpy(2 * m).cuda(), torch.from_numpy(2 * v).cuda()
    print("roots from 2^%d, t=%d" % (exponent, t), flush=True)
    P.fl_adamw_step(lay, hp, t, g, p, dm, dv, None)
    assert np.array_equal(dv.cpu().numpy(), v) and np.array_equal(dm.cpu().numpy(), m)
    assert np.array_equal(p.cpu().numpy(), -(lr * want))
    lay.close()


def test_root_over_its_whole_range(env):
    """The same quotients for every float from 2^-100 to 2^60, the roots and
    quotients of the reference rounded from double (which is exact for both)."""
    torch, P, _ = env
    hp = dict(lr=1.0, beta1=0.5, beta2=0.5, eps=2.0 ** -60, weight_decay=0.0)
    n = 1 << 24
    lay = P.Layout(np.array([0, n], np.int64), np.ones(1, np.uint8))
    g, mantissas = torch.zeros(n, device="cuda"), torch.arange(n, dtype=torch.int32, device="cuda")
    print("roots from 2^-100 to 2^60", flush=True)
    for exponent in range(-100, 60, 2):
        v = (mantissas + ((exponent + 127) << 23)).view(torch.float32)
        den = v.double().sqrt().float() + 2.0 ** -60
        m = den * (1.0 - 2.0 ** -21)
        p, dm, dv = torch.zeros(n, device="cuda"), 2 * m, 2 * v
        P.fl_adamw_step(lay, hp, 1000, g, p, dm, dv, None)
        assert torch.equal(dv, v) and torch.equal(dm, m)
        assert torch.equal(p, -(m.double() / den.double()).float()), exponent
    lay.close()
