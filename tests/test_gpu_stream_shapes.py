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


# 256 CUs x 512 elements a unit: 20, 100 and 384 units per CU, each with a
# length just inside and a ragged one just past it.
@pytest.mark.parametrize("n", [u * 131072 + d for u in (20, 100, 384) for d in (0, 131072 + 3)])
def test_launch_bands(env, n):
    torch, P, orc = env
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
    P.fl_local_step(lay, ADAMW, 3, peers, 1.0 / 3, master, m, v, work)
    orc.adamw_step(off, dec, ADAMW, 3, want, rm, r1, r2, rw)
    H.assert_state_parity("step", dict(master=master.cpu().numpy(), m=m.cpu().numpy(),
                                       v=v.cpu().numpy(), working=H.to_u16(work)),
                          dict(master=rm, m=r1, v=r2, working=rw), bitwise=True)
    lay.close()
