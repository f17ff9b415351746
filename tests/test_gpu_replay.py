"""GPU parity: the replay verbs against the oracle, element by element, on small and ragged shapes."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import assert_close, assert_sample_equal, check_gpu_tree, dev, host

pytestmark = pytest.mark.gpu
F32 = np.float32
U64 = 1 << 64


def make_pair(C, P, ob, ab, **kw):
    from paper_1803_00933_amd import apex
    return apex.Replay(C, P, ob, ab, **kw), oracle.Replay(C, P, ob, ab, **kw)


def add_both(g, o, rng, cnt, dist=lambda rng, n: rng.lognormal(0, 1, n)):
    from paper_1803_00933_amd import apex
    obs = rng.integers(0, 256, (cnt, o.obs_bytes), dtype=np.uint8)
    act = rng.integers(0, 256, (cnt, o.act_bytes), dtype=np.uint8)
    ret, gacc = rng.standard_normal(cnt).astype(F32), rng.random(cnt).astype(F32)
    prio = dist(rng, cnt).astype(F32)
    rco, fo = o.add(prio, obs, act, ret, gacc)
    rcg, fg = g.add(dev(prio), dev(obs), dev(act), dev(ret), dev(gacc))
    assert rcg == rco
    if rco == 0:
        assert fg == fo
    return rco


def sample_both(g, o, rng, nb, k, beta=0.4, rnd=None):
    rnd = rng.integers(0, U64, nb * k, dtype=np.uint64) if rnd is None else rnd
    rco, oo = o.sample(nb, k, beta, rnd)
    rcg, go = g.sample(nb, k, beta, dev(rnd))
    assert rcg == rco
    if rco == 0:
        torch.cuda.synchronize()
        assert_sample_equal(go, oo)
    return oo


@pytest.mark.parametrize("P,C,ob,ab", [
    (100, 80, 32, 4),            # one tree level, everything in LDS
    (8192, 4096, 32, 4),         # two levels
    (5000, 4000, 12, 8),         # ragged level sizes, dword copy path
    (300_000, 250_000, 7, 3),    # three levels with ragged tails, byte copy path
    (70_000, 65_000, 4112, 32),  # long-row copy path with a partial last chunk
])
def test_random_operation_sequences(P, C, ob, ab):
    rng = np.random.default_rng(P)
    g, o = make_pair(C, P, ob, ab)
    pareto = lambda rng, n: np.where(rng.random(n) < 0.2, 0.0, rng.pareto(1.1, n) + 1.0)
    for it in range(12):
        cnt = int(rng.integers(1, max(2, P // 4)))
        if o.size + cnt > P:
            assert add_both(g, o, rng, cnt) == oracle.ERR_FULL
            cnt = P - o.size
        if cnt:
            assert add_both(g, o, rng, cnt, pareto if it % 2 else (lambda r, n: r.lognormal(0, 2, n))) == 0
        check_gpu_tree(g, o)
        for nb, k in ((1, 32), (3, 50), (1, 1), (2, 257)):
            oo = sample_both(g, o, rng, nb, k, beta=float(rng.uniform(0, 1)))
        # learner feedback: the sampled keys (with their repeats), some stale and some future keys
        keys = np.concatenate([oo["key"], rng.integers(0, max(1, o.head), 5).astype(np.uint64),
                               np.array([o.tail, o.tail + 7, U64 - 1], np.uint64), oo["key"][:40]])
        newp = pareto(rng, len(keys)).astype(F32)
        newp[:3] = [np.nan, np.inf, 1e30]
        assert o.update_priorities(keys, newp) == 0
        assert g.update_priorities(dev(keys), dev(newp)) == 0
        check_gpu_tree(g, o)
        rco, eo = o.evict()
        rcg, eg = g.evict()
        assert (rcg, eg) == (rco, eo)
        check_gpu_tree(g, o)
        sample_both(g, o, rng, 2, 64)


@pytest.mark.parametrize("P", [512, 513, 1024, 1025, 4608, 4609, 32_768, 32_769, 65_536, 65_537, 294_912, 294_913])
def test_tree_shapes_around_the_summit(P):
    """Sizes on both sides of every border of the tree's shape: the level that walks start from is the leaves themselves
    (512 in one read, 513 and 1024 in two), a summit of 4 and 16 children per node (1025, 4608; 65,537 and 294,912 above
    more levels), or an ordinary level (32,768 in one read, 32,769 and 65,536 in two).  Rounds that wrap around the ring
    and cross several workgroups, draws at the very ends of the cumulative mass, updates and evictions, bit for bit
    against the oracle."""
    rng = np.random.default_rng(P)
    C = P * 3 // 4
    g, o = make_pair(C, P, 16, 4)
    assert add_both(g, o, rng, C) == 0
    for it in range(5):
        cnt = min(P - o.size, (1, 700, 2100, 63, 5000)[it])
        assert add_both(g, o, rng, cnt) == 0
        check_gpu_tree(g, o)
        edges = np.array([0, U64 - 1] * 8, np.uint64)
        sample_both(g, o, rng, 1, 16, rnd=edges)
        for nb, k in ((1, 1), (2, 17), (5, 450)):     # batches that leave a wave's four samples incomplete
            oo = sample_both(g, o, rng, nb, k)
        pr = rng.lognormal(0, 2, len(oo["key"])).astype(F32)
        assert g.update_priorities(dev(oo["key"]), dev(pr)) == o.update_priorities(oo["key"], pr) == 0
        assert g.evict() == o.evict()
        check_gpu_tree(g, o)
        sample_both(g, o, rng, 3, 64)


@pytest.mark.parametrize("ob,ab,nb,k", [
    (1, 1, 1, 32), (15, 3, 1, 33), (16, 4, 2, 31), (17, 5, 3, 64), (67 * 4, 21 * 4, 1, 256), (2048, 64, 1, 100),
    (2049, 65, 2, 65), (4095, 130, 1, 200), (4096, 2, 1, 32), (4097, 7, 1, 40),       # row lengths and action bytes
    (24, 4, 1, 2048), (24, 4, 1, 2049), (20, 4, 1, 4096), (20, 4, 2, 4097), (12, 8, 700, 3),  # batch sizes and counts
    (1024, 4, 1, 2049), (1025, 4, 1, 2049), (7, 3, 1, 3000), (24, 4, 2, 2049),
])
def test_sample_in_one_launch(ob, ab, nb, k):
    """replay.Sample of short rows as one launch, at the edges of what its lanes and workgroups hold: rows and action
    bytes around every width they are copied in, batches around the borders between one workgroup, several (tickets)
    and a launch of their own for the weights.  Called twice in a row (the tickets are back at 0) and on the memory
    with prioritized eviction too."""
    from paper_1803_00933_amd import apex
    rng = np.random.default_rng(ob * 7 + k)
    g, o = make_pair(3000, 4000, ob, ab)
    assert add_both(g, o, rng, 3000) == 0
    for _ in range(2):
        sample_both(g, o, rng, nb, k)
    gp = apex.PeReplay(3000, 4000, ob, ab)
    op = oracle.PrioritizedEvictionReplay(3000, 4000, ob, ab)
    obs = rng.integers(0, 256, (2000, ob), dtype=np.uint8)
    act = rng.integers(0, 256, (2000, ab), dtype=np.uint8)
    ret, gacc, prio = (rng.random(2000).astype(F32) for _ in range(3))
    assert op.add(prio, obs, act, ret, gacc)[0] == 0
    assert gp.add(dev(prio), dev(obs), dev(act), dev(ret), dev(gacc)) == 0
    for _ in range(2):
        sample_both(gp, op, rng, nb, k)


@pytest.mark.parametrize("ob,ab,nb,k", [
    (16, 1, 384, 1), (16, 2, 1, 384), (17, 3, 1, 385), (31, 4, 12, 32), (32, 5, 11, 33), (100, 255, 6, 64), (100, 257, 1, 65),
    (2047, 4, 2, 192), (2048, 4, 3, 512), (2048, 4, 1, 513), (4095, 4, 1, 1023), (4096, 4, 1, 1024),       # lines of the rule
    (4097, 4, 1, 1024), (4100, 4, 1, 1025), (8207, 4, 1, 1), (8207, 4, 48, 32), (8207, 4, 47, 33),
    (28224, 4, 3, 333), (30720, 4, 1, 600), (30721, 4, 1, 300), (61441, 4, 1, 200), (70000, 4, 1, 700),  # pieces per lane
])
@pytest.mark.parametrize("P", [900, 40_000])     # one level of tree, two with a wide top
def test_sample_with_a_workgroup_per_sample(P, ob, ab, nb, k):
    """Around the lines where replay.Sample changes between a workgroup per sample, 16 lanes per sample and two launches,
    in turn with calls of the other kinds on the same tickets."""
    if P * ob > 1 << 28:
        P = 2000
    rng = np.random.default_rng(ob + k)
    g, o = make_pair(P - 50, P, ob, ab)
    assert add_both(g, o, rng, P - 60) == 0 and add_both(g, o, rng, 50) == 0 and g.evict() == o.evict()
    for n in (nb, 1, nb, nb):
        sample_both(g, o, rng, n, k)
        sample_both(g, o, rng, 2, 40)
    if ob < 100:
        sample_both(g, o, rng, 3, 700)
    sample_both(g, o, rng, nb, k)
    torch.cuda.synchronize()
    assert int(g.scratch[256:256 + 1024 * 16 * 4].view(torch.int32).abs().max()) == 0


@pytest.mark.parametrize("P", [1025, 4608, 70_000, 294_912])
@pytest.mark.parametrize("m", [512, 513, 1024])
def test_updates_on_trees_with_a_summit(P, m):
    """Batches of half to the whole of a workgroup on trees with a summit and without one: random keys, the keys of a batch,
    one key again and again, stale ones; given priorities and those of the learner's Q-values."""
    rng = np.random.default_rng(P + m)
    g, o = make_pair(P - 200, P, 16, 4)
    assert add_both(g, o, rng, P - 200) == 0 and add_both(g, o, rng, 150) == 0
    assert g.evict() == o.evict()
    for keys in (rng.integers(0, o.tail + 50, m), sample_both(g, o, rng, 1, m)["key"], np.full(m, o.head + 5)):
        keys, pr = keys.astype(np.uint64), rng.lognormal(0, 2, m).astype(F32)
        assert g.update_priorities(dev(keys), dev(pr)) == o.update_priorities(keys, pr) == 0
        check_gpu_tree(g, o)
        q = [rng.standard_normal(shape).astype(F32) for shape in (m, (m, 3), (m, 3))]
        p_out = torch.empty(m, dtype=torch.float32, device="cuda:0")
        rc, p_ref = o.update_from_q(keys, *q)
        assert g.update_from_q(dev(keys), *(dev(x) for x in q), p_out) == rc == 0
        assert np.array_equal(host(p_out).view(np.uint32), p_ref.view(np.uint32))
        check_gpu_tree(g, o)
    sample_both(g, o, rng, 1, m)


@pytest.mark.parametrize("m", [1, 63, 64, 65, 255, 257, 1023, 1024, 1025, 1087, 2047, 2048, 2049, 2112, 4095, 4096, 4097])
@pytest.mark.parametrize("A", [1, 2, 3, 9, 18])
def test_updates_at_the_edges_of_their_workgroups(m, A):
    """Updates of any number of pairs around the workgroups' shares and the line between one launch and two: repeats
    across the shares (the last one wins), stale keys at both ends, given priorities and the learner's, with ties of the
    greedy action and Q-values that compare with nothing."""
    rng = np.random.default_rng(100 * m + A)
    g, o = make_pair(3000, 4097, 16, 4)
    assert add_both(g, o, rng, 3000) == 0 and add_both(g, o, rng, 1000) == 0
    assert g.evict() == o.evict()                        # valid keys: [1000, 4000)
    for distinct in (3, 400, 3100):                      # few keys often, many once, some stale
        keys = (950 + rng.integers(0, distinct, m)).astype(np.uint64)
        keys[rng.random(m) < 0.5] += np.uint64(60)
        pr = rng.lognormal(0, 1, m).astype(F32)
        assert g.update_priorities(dev(keys), dev(pr)) == o.update_priorities(keys, pr) == 0
        check_gpu_tree(g, o)
        q_on = np.round(rng.standard_normal((m, A)) * 2).astype(F32) / 2
        q_on[rng.random((m, A)) < 0.1] = np.nan
        q_on[rng.random(m) < 0.1] = -np.inf
        q = [rng.standard_normal(m).astype(F32), q_on, rng.standard_normal((m, A)).astype(F32)]
        p_out = torch.empty(m, dtype=torch.float32, device="cuda:0")
        rc, p_ref = o.update_from_q(keys, *q)
        assert g.update_from_q(dev(keys), *(dev(x) for x in q), p_out) == rc == 0
        assert np.array_equal(host(p_out).view(np.uint32), p_ref.view(np.uint32))
        check_gpu_tree(g, o)


@pytest.mark.parametrize("obs_bytes", [1, 3, 4, 12, 15, 16, 17, 100, 128, 255, 256, 257])
@pytest.mark.parametrize("act_bytes", [1, 16, 17])
def test_adds_of_short_rows_in_one_launch(obs_bytes, act_bytes):
    """Whole adds around the lines between one launch and two and the edges of the workgroups and passes, from aligned and
    misaligned rows, over the end of the ring."""
    rng = np.random.default_rng(obs_bytes)
    P = 21_000
    g, o = make_pair(1000, P, obs_bytes, act_bytes)
    for it, cnt in enumerate((1, 64, 127, 129, 255, 256, 257, 1023, 2100, 16_384, 16_385, 3000, 20_000, 700)):
        obs, act = (rng.integers(0, 256, (cnt, n), dtype=np.uint8) for n in (obs_bytes, act_bytes))
        ret, gacc, prio = rng.standard_normal(cnt).astype(F32), rng.random(cnt).astype(F32), rng.lognormal(0, 1, cnt).astype(F32)
        d_obs = torch.empty(cnt * obs_bytes + 16, dtype=torch.uint8, device="cuda:0")[it % 3:][:cnt * obs_bytes].view(cnt, obs_bytes)
        d_obs.copy_(dev(obs))
        rc, first = g.add(dev(prio), d_obs, dev(act), dev(ret), dev(gacc))
        assert (rc, first) == o.add(prio, obs, act, ret, gacc) and rc == 0
        rows = (first + np.arange(cnt)) % P
        torch.cuda.synchronize()
        assert np.array_equal(host(g.obs_view()).reshape(P, obs_bytes)[rows], obs)
        assert np.array_equal(host(g.act_view()).reshape(P, act_bytes)[rows], act)
        assert np.array_equal(host(g.ret_view())[rows], ret) and np.array_equal(host(g.gacc_view())[rows], gacc)
        check_gpu_tree(g, o)
        assert g.evict() == o.evict()
    check_gpu_tree(g, o)
    full = dev(np.zeros((P, obs_bytes), np.uint8))
    assert g.add(dev(np.ones(P, F32)), full)[0] == oracle.ERR_FULL and g.add(dev(np.ones(0, F32)), full[:0]) == (0, o.tail)
    check_gpu_tree(g, o)


@pytest.mark.parametrize("P", [3000, 100_000])
def test_adds_and_evictions_at_the_edges_of_their_workgroups(P):
    """Rounds of one wave, of whole and ragged workgroups and just beyond the largest one, each evicted again."""
    rng = np.random.default_rng(P)
    C = P - 1100
    g, o = make_pair(C, P, 16, 4)
    assert add_both(g, o, rng, C) == 0
    for cnt in (1, 63, 64, 65, 128, 129, 191, 1023, 1024, 1025):
        assert add_both(g, o, rng, cnt) == 0
        check_gpu_tree(g, o)
        assert g.evict() == o.evict() == (0, cnt)
        check_gpu_tree(g, o)
    sample_both(g, o, rng, 1, 256)


@pytest.mark.parametrize("prioritized_eviction", [False, True])
def test_sample_recovers_from_stale_tickets(prioritized_eviction):
    """Sample calls that overlapped although they must be ordered can leave the tickets of the weights at any value
    (planted here, in every word): after two more calls with weights from several workgroups, every later one is right
    again, whatever calls without tickets or of fewer batches lie in between."""
    from paper_1803_00933_amd import apex
    rng = np.random.default_rng(8)
    if prioritized_eviction:
        g, o = apex.PeReplay(3000, 4000, 32, 4), oracle.PrioritizedEvictionReplay(3000, 4000, 32, 4)
        prio = rng.random(3000).astype(F32)
        obs, act = (rng.integers(0, 256, (3000, n), dtype=np.uint8) for n in (32, 4))
        assert o.add(prio, obs, act, prio, prio)[0] == 0
        assert g.add(dev(prio), dev(obs), dev(act), dev(prio), dev(prio)) == 0
    else:
        g, o = make_pair(3000, 4000, 32, 4)
        assert add_both(g, o, rng, 3000) == 0
    words = g.scratch[256:256 + 1024 * 16 * 4].view(torch.int32)   # behind the device state: 16 words per batch
    assert int(words.abs().max()) == 0
    sample_both(g, o, rng, 3, 40)
    words.fill_(1000)                 # no launch below has as many workgroups per batch
    for nb in (3, 1):
        assert g.sample(nb, 512, 0.4, dev(rng.integers(0, U64, nb * 512, dtype=np.uint64)))[0] == 0
    for nb, k in ((1, 512), (1, 33), (1, 512), (1, 512), (3, 200), (1, 32), (1, 32), (1, 32), (3, 512), (2, 4096), (3, 2048)):
        sample_both(g, o, rng, nb, k)
    assert int(words.view(1024, 16)[:3, :4].abs().max()) == 0


@pytest.mark.parametrize("ob", [12, 15, 16, 17, 31, 100, 1028, 1039, 4096, 4097, 5003, 8207, 32772])
def test_rows_of_any_length_at_any_alignment(ob):
    """Observation rows around the edges of the 16-byte pieces, of a launch's share of a row and of the short and long
    row kernels, from and to addresses that divide by nothing: add, gather, sample, and the pipeline's steps."""
    from paper_1803_00933_amd import apex
    rng = np.random.default_rng(ob)
    g, o = make_pair(2100, 2500, ob, 3)
    for n in (1100, 1000):                                   # (from 1024 long rows on they are copied as one run)
        prio = rng.lognormal(0, 1, n).astype(F32)
        obs, act = rng.integers(0, 256, (n, ob), dtype=np.uint8), rng.integers(0, 256, (n, 3), dtype=np.uint8)
        ret, gacc = rng.standard_normal(n).astype(F32), rng.random(n).astype(F32)
        assert o.add(prio, obs, act, ret, gacc)[0] == 0
        shifted = torch.empty(n * ob + 1, dtype=torch.uint8, device="cuda:0")[1:].view(n, ob)
        shifted.copy_(torch.from_numpy(obs))
        assert g.add(dev(prio), shifted, dev(act), dev(ret), dev(gacc))[0] == 0
    sample_both(g, o, rng, 2, 77)
    rnd = rng.integers(0, U64, 70, dtype=np.uint64)
    oo = o.sample(1, 70, 0.4, rnd)[1]
    for shift in (0, 1):
        buf = torch.full((70 * ob + 3,), 255, dtype=torch.uint8, device="cuda:0")
        to = buf[shift:shift + 70 * ob].view(70, ob)
        assert g.gather(dev(oo["slot"].astype(np.uint32)), obs=to) == 0
        torch.cuda.synchronize()
        assert np.array_equal(host(to), oo["obs"])
        assert bool((buf[shift + 70 * ob:] == 255).all()) and bool((buf[:shift] == 255).all())
    pipe = apex.Pipeline(g, 3, 1, 70)
    rnd, newp = rng.integers(0, U64, (3, 70), dtype=np.uint64), rng.lognormal(0, 1, (3, 70)).astype(F32)
    d_rnd, d_newp = dev(rnd), dev(newp)
    assert pipe.fork() == 0 and pipe.steps(3, 0.4, d_rnd, d_newp)[0] == 0 and pipe.join() == 0
    torch.cuda.synchronize()
    for s in range(3):
        oo = o.sample(1, 70, 0.4, rnd[s])[1]
        o.update_priorities(oo["key"], newp[s])
        assert_sample_equal(pipe.sets[s], oo)
    check_gpu_tree(g, o)
    pipe.close()


@pytest.mark.parametrize("P,C,ob,ab", [(5000, 4000, 48, 8), (3000, 2500, 4112, 4)])
def test_add_with_payload_written_in_place(P, C, ob, ab):
    """A producer writes observations and actions of the coming keys straight into the ring (row
    (tail + i) mod P of each column) and adds with NULL for those columns: same memory as a copying add."""
    rng = np.random.default_rng(P + ob)
    g, o = make_pair(C, P, ob, ab)
    for it in range(7):     # wraps around the ring
        cnt = int(rng.integers(1, P - o.size + 1)) if o.size < P else 0
        if cnt:
            obs = rng.integers(0, 256, (cnt, ob), dtype=np.uint8)
            act = rng.integers(0, 256, (cnt, ab), dtype=np.uint8)
            ret, gacc = rng.standard_normal(cnt).astype(F32), rng.random(cnt).astype(F32)
            prio = rng.lognormal(0, 1, cnt).astype(F32)
            rows = torch.from_numpy(((o.tail + np.arange(cnt)) % P).astype(np.int64)).cuda()
            g.obs_view().index_copy_(0, rows, dev(obs))
            g.act_view().index_copy_(0, rows, dev(act))
            assert o.add(prio, obs, act, ret, gacc)[0] == 0
            rc, first = g.add(dev(prio), None, None, dev(ret), dev(gacc))
            assert (rc, first) == (0, o.tail - cnt)
        check_gpu_tree(g, o)
        sample_both(g, o, rng, 2, 96)
        assert g.evict() == o.evict()
    sample_both(g, o, rng, 8, 500)      # the payload of most live keys, as the oracle stored it


def test_large_update_batches_with_heavy_duplication():
    # more than one workgroup's worth of pairs: the two-pass path; few distinct keys: many repeats
    rng = np.random.default_rng(10)
    g, o = make_pair(20_000, 20_000, 16, 4)
    add_both(g, o, rng, 20_000)
    for m, distinct in ((1025, 50), (8192, 300), (5000, 20_000), (1024, 3), (64, 1)):
        keys = rng.integers(0, distinct, m).astype(np.uint64)
        newp = rng.lognormal(0, 1, m).astype(F32)
        assert o.update_priorities(keys, newp) == 0
        assert g.update_priorities(dev(keys), dev(newp)) == 0
        check_gpu_tree(g, o)
    sample_both(g, o, rng, 16, 512)


def test_gather_by_slot():
    rng = np.random.default_rng(9)
    for ob, ab in ((28224, 4), (64, 4), (256, 32), (10, 6)):
        g, o = make_pair(900, 1000, ob, ab)
        add_both(g, o, rng, 950)
        oo = sample_both(g, o, rng, 1, 300)
        out = g.alloc_sample_outputs(1, 300)
        slot = dev(oo["slot"])
        assert g.gather(slot, out["obs"], out["act"], out["ret"], out["gacc"]) == 0
        torch.cuda.synchronize()
        for name in ("obs", "act", "ret", "gacc"):
            assert np.array_equal(host(out[name]), oo[name]), name
        assert g.gather(slot[:0]) == 0


def test_extreme_uniforms_and_edges():
    rng = np.random.default_rng(1)
    g, o = make_pair(6000, 6000, 16, 4)
    add_both(g, o, rng, 6000)
    for fill in (0, U64 - 1, 1 << 63):
        sample_both(g, o, rng, 2, 100, rnd=np.full(200, fill, np.uint64))
    sample_both(g, o, rng, 1, 9000)                      # more samples than transitions
    sample_both(g, o, rng, 1, 65536 // 2)
    # all mass on one transition
    g2, o2 = make_pair(5000, 5000, 16, 4, alpha=1.0, eps=0.0)
    add_both(g2, o2, rng, 5000, lambda r, n: np.where(np.arange(n) == 4321, 1e6, 0.0))
    oo = sample_both(g2, o2, rng, 1, 64)
    assert (oo["slot"] == 4321).sum() >= 63


def test_alpha_zero_and_beta_edges():
    rng = np.random.default_rng(2)
    g, o = make_pair(10_000, 10_000, 16, 4, alpha=0.0)
    add_both(g, o, rng, 10_000)
    oo = sample_both(g, o, rng, 4, 128)
    assert np.all(oo["weight"] == 1.0)
    g, o = make_pair(10_000, 10_000, 16, 4)
    add_both(g, o, rng, 10_000)
    for beta in (0.0, 1.0, 0.4):
        sample_both(g, o, rng, 2, 512, beta=beta)


def test_status_codes():
    from paper_1803_00933_amd import apex
    rng = np.random.default_rng(3)
    g, o = make_pair(100, 128, 16, 4, min_size_to_sample=50)
    rnd = dev(np.zeros(8, np.uint64))
    assert g.sample(1, 8, 0.4, rnd)[0] == apex.ERR_NOT_READY == o.sample(1, 8, 0.4, np.zeros(8, np.uint64))[0]
    add_both(g, o, rng, 49)
    assert g.sample(1, 8, 0.4, rnd)[0] == apex.ERR_NOT_READY
    add_both(g, o, rng, 1)
    assert g.sample(1, 8, 0.4, rnd)[0] == apex.OK
    g2, o2 = make_pair(100, 128, 16, 4)
    assert g2.sample(1, 8, 0.4, rnd)[0] == apex.ERR_EMPTY == o2.sample(1, 8, 0.4, np.zeros(8, np.uint64))[0]
    assert g.sample(0, 8, 0.4, rnd)[0] == apex.ERR_INVALID_ARG
    assert g.sample(1, 0, 0.4, rnd)[0] == apex.ERR_INVALID_ARG
    assert g.sample(1, 8, -1.0, rnd)[0] == apex.ERR_INVALID_ARG
    big = dev(np.zeros(8, np.uint64))
    assert apex.lib.apex_replay_sample(g.h, 2, 40000, 0.4, big.data_ptr(), None, big.data_ptr(), *([None] * 6)) \
        == apex.ERR_TOO_LARGE
    assert apex.lib.apex_replay_sample(g.h, 1, 8, 0.4, big.data_ptr(), None, None, *([None] * 6)) == apex.ERR_INVALID_ARG
    assert g.evict() == (0, 0) and g.add(dev(np.zeros(0, F32)))[0] == apex.OK
    assert g.update_priorities(dev(np.zeros(0, np.uint64)), dev(np.zeros(0, F32))) == apex.OK
    torch.cuda.synchronize()
    check_gpu_tree(g, o)


@pytest.mark.parametrize("P,C", [(128, 100), (1 << 20, 1_000_000)])   # the larger shape has a top level of 256 nodes
def test_fused_steps_refuse_an_empty_or_unready_memory(P, C):
    """Learner steps as one launch each obey the same gate as apex_replay_sample: nothing stored -> EMPTY, fewer
    than min_size_to_sample -> NOT_READY, with or without priorities to write back, and nothing is enqueued
    (tree, counters and buffers stay as they were)."""
    from paper_1803_00933_amd import apex
    rng = np.random.default_rng(17)
    k = 8
    rnd, newp = dev(rng.integers(0, U64, (3, k), dtype=np.uint64)), dev(rng.random((3, k)).astype(F32))
    for min_size, fill, want in ((0, 0, apex.ERR_EMPTY), (50, 0, apex.ERR_NOT_READY), (50, 49, apex.ERR_NOT_READY)):
        g, o = make_pair(C, P, 16, 4, min_size_to_sample=min_size)
        if fill:
            assert add_both(g, o, rng, fill) == 0
        pipe = apex.Pipeline(g, 4, 1, k)
        for s_ in pipe.sets:
            s_["slot"].fill_(-7)
        torch.cuda.synchronize()
        before = g.stats()
        assert o.sample(1, k, 0.4, np.zeros(k, np.uint64))[0] == want
        assert pipe.fork() == 0
        assert pipe.steps(3, 0.4, rnd, newp)[0] == want
        assert pipe.steps(3, 0.4, rnd, None)[0] == want
        assert pipe.join() == 0
        torch.cuda.synchronize()
        assert g.stats() == before
        assert all(int((s_["slot"] != -7).sum()) == 0 for s_ in pipe.sets)
        check_gpu_tree(g, o)
        if fill:                                   # one more transition and the same call goes through
            assert add_both(g, o, rng, 1) == 0
            assert pipe.fork() == 0
            rc, first = pipe.steps(3, 0.4, rnd, newp)
            assert rc == apex.OK and pipe.join() == 0
            torch.cuda.synchronize()
            for i in range(3):
                rco, oo = o.sample(1, k, 0.4, host(rnd[i], np.uint64))
                assert rco == 0 and o.update_priorities(oo["key"], host(newp[i])) == 0
                assert_sample_equal(pipe.sets[(first + i) % 4], oo)
            check_gpu_tree(g, o)
        pipe.close()


def test_tiny_workload_full_trace():
    """The small configuration end to end: 200 rounds of {n-step priorities, add 400, sample 32,
    update with fresh |N(0,1)| errors, evict}; every output of every round is compared."""
    from paper_1803_00933_amd import apex, synth
    w = synth.WORKLOADS["tiny"]
    g, o = make_pair(w.capacity, w.max_slots, w.obs_bytes, w.act_bytes, alpha=w.alpha, eps=w.eps, frac_bits=w.frac_bits)
    key0 = 0
    for rnd_i in range(200):
        d = synth.actor_round(w, rnd_i)
        ref = oracle.nstep_priorities(d["q_online"], d["q_target"], d["action"], d["reward"], d["discount"],
                                      w.n, w.alpha, w.eps, w.frac_bits, w.max_slots)
        rc, prio, ret, gacc, fx = apex.nstep_priorities(dev(d["q_online"]), dev(d["q_target"]), dev(d["action"]),
                                                        dev(d["reward"]), dev(d["discount"]), w.n, w.alpha, w.eps,
                                                        w.frac_bits, w.max_slots)
        assert rc == 0
        obs = synth.obs_rows(w.seed, key0, w.add_count, w.obs_bytes)
        rco, fo = o.add(ref[0].reshape(-1), obs, d["act"], ref[1].reshape(-1), ref[2].reshape(-1))
        rcg, fg = g.add(prio.view(-1), dev(obs), dev(d["act"]), ret.view(-1), gacc.view(-1))   # device to device
        assert (rcg, fg) == (rco, fo) == (0, key0)
        key0 += w.add_count
        torch.cuda.synchronize()
        assert np.array_equal(host(fx, np.uint64), ref[3])
        rnd = synth.uniforms(w.seed, rnd_i, 1, w.k).reshape(-1)
        rco, oo = o.sample(1, w.k, w.beta, rnd)
        rcg, go = g.sample(1, w.k, w.beta, dev(rnd))
        assert rcg == rco == 0
        torch.cuda.synchronize()
        assert_sample_equal(go, oo)
        assert np.array_equal(oo["obs"], np.concatenate([synth.obs_rows(w.seed, int(kk), 1, w.obs_bytes)
                                                         for kk in oo["key"]]))
        newp = synth.priorities(w.td_dist, w.seed, rnd_i, w.k)
        assert o.update_priorities(oo["key"], newp) == 0
        assert g.update_priorities(go["key"], dev(newp)) == 0
        assert g.evict() == o.evict()
        if rnd_i % 10 == 9 or rnd_i < 12:
            st = check_gpu_tree(g, o)
            assert st["size"] == min(key0, w.capacity)
    check_gpu_tree(g, o)


def test_split_calls_on_separate_streams():
    """sample_begin / sample_finish and add_payload / add_publish, tree work and copies on different
    streams ordered by events, against the oracle's plain sequence."""
    rng = np.random.default_rng(12)
    C, P, ob, ab, k, cnt = 3000, 4096, 28224, 4, 128, 500
    g, o = make_pair(C, P, ob, ab)
    add_both(g, o, rng, C)
    tree_s, copy_s = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    outs, refs = [], []
    for step in range(8):
        out = g.alloc_sample_outputs(1, k)
        out["mass"] = torch.empty(k, dtype=torch.int64, device="cuda:0")
        rnd = rng.integers(0, U64, k, dtype=np.uint64)
        newp = rng.lognormal(0, 1, k).astype(F32)
        obs = rng.integers(0, 256, (cnt, ob), dtype=np.uint8)
        act = rng.integers(0, 256, (cnt, ab), dtype=np.uint8)
        ret, gacc, prio = (rng.standard_normal(cnt).astype(F32) for _ in range(3))
        d = [dev(x) for x in (rnd, newp, obs, act, ret, gacc, prio)]
        torch.cuda.synchronize()
        # oracle: sample, update, add, evict
        rco, oo = o.sample(1, k, 0.4, rnd)
        o.update_priorities(oo["key"], newp)
        o.add(prio, obs, act, ret, gacc)
        o.evict()
        # device: the payload copy of the add runs beside the learner step
        assert g.add_payload(cnt, d[2], d[3], d[4], d[5], stream=copy_s) == 0
        payload_done = torch.cuda.Event()
        payload_done.record(copy_s)
        assert g.sample_begin(1, k, d[0], out, stream=tree_s) == 0
        drawn = torch.cuda.Event()
        drawn.record(tree_s)
        copy_s.wait_event(drawn)
        assert g.sample_finish(1, k, 0.4, out, stream=copy_s) == 0
        assert g.update_priorities(out["key"], d[1], stream=tree_s) == 0
        tree_s.wait_event(payload_done)
        assert g.add_publish(d[6], stream=tree_s)[0] == 0
        assert g.evict(stream=tree_s)[0] == 0
        gathered = torch.cuda.Event()
        gathered.record(copy_s)
        tree_s.wait_event(gathered)          # the next payload must not overwrite rows still being read
        copy_s.wait_stream(tree_s)           # and needs the advanced tail
        outs.append(out), refs.append(oo)
    torch.cuda.synchronize()
    for out, oo in zip(outs, refs):
        assert_sample_equal(out, oo)
        assert np.array_equal(host(out["mass"], np.uint64), oo["mass"])
    check_gpu_tree(g, o)


def test_captured_launches_replay_correctly():
    """A captured sequence of add / sample / update / evict is replayed several times, with eager work
    and synchronisations in between; every replay is checked against the oracle doing the same."""
    rng = np.random.default_rng(13)
    C, P, ob, ab, k, cnt = 1000, 2048, 64, 4, 64, 100
    g, o = make_pair(C, P, ob, ab)
    add_both(g, o, rng, C)
    rnd = [rng.integers(0, U64, k, dtype=np.uint64) for _ in range(3)]
    newp = [rng.lognormal(0, 1, k).astype(F32) for _ in range(3)]
    obs = rng.integers(0, 256, (cnt, ob), dtype=np.uint8)
    act = rng.integers(0, 256, (cnt, ab), dtype=np.uint8)
    ret, gacc, prio = (rng.standard_normal(cnt).astype(F32) for _ in range(3))
    d_rnd, d_newp = [dev(x) for x in rnd], [dev(x) for x in newp]
    d_obs, d_act, d_ret, d_gacc, d_prio = (dev(x) for x in (obs, act, ret, gacc, prio))
    outs = [g.alloc_sample_outputs(1, k) for _ in range(3)]

    def sequence():
        assert g.add(d_prio, d_obs, d_act, d_ret, d_gacc)[0] == 0
        for i in range(3):
            assert g.sample(1, k, 0.4, d_rnd[i], out=outs[i])[0] == 0
            assert g.update_priorities(outs[i]["key"], d_newp[i]) == 0
        assert g.evict() == (0, cnt)

    def oracle_sequence():
        o.add(prio, obs, act, ret, gacc)
        res = []
        for i in range(3):
            res.append(o.sample(1, k, 0.4, rnd[i])[1])
            o.update_priorities(res[-1]["key"], newp[i])
        assert o.evict() == (0, cnt)
        return res

    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s):
        sequence()
    for replay in range(4):
        graph.replay()
        torch.cuda.synchronize()
        res = oracle_sequence()
        for i in range(3):
            assert_sample_equal(outs[i], res[i])
        assert g.resync() == 0
        check_gpu_tree(g, o)
        if replay == 1:                      # eager work between replays, on the same memory
            add_both(g, o, rng, 50)
            sample_both(g, o, rng, 1, 32)
            assert g.evict() == o.evict()
            assert g.resync() == 0


# One batch per step of 16-byte-aligned rows is one launch per step; 8 x 288 samples per step is above the
# size from which the pipeline sends a step's gather to its copy stream.
# (batches per step, k, observation bytes).  Rows of at most 1 KB make a small add round one launch
# (n-step priorities, payload and masses together), issued by add_end.
PIPELINE_STEP_SHAPES = [(1, 96, 4224), (8, 288, 4224), (1, 64, 256), (1, 64, 100), (1, 32, 7), (1, 32, 1001)]


@pytest.mark.parametrize("depth", [3, 2])      # two buffer sets: too few for the one-launch step, two launches instead
@pytest.mark.parametrize("nb,k,ob", PIPELINE_STEP_SHAPES)
def test_pipeline_matches_the_plain_call_order(nb, k, ob, depth):
    """apex_pipeline_*: learner steps (for steps of several batches: with the gathers on the second
    stream) and add rounds whose payload copy runs beside them, against the oracle doing draw, update,
    [add], [evict] one after the other."""
    from paper_1803_00933_amd import apex, synth
    w = synth.WORKLOADS["tiny"].scaled(obs_bytes=ob, capacity=3000, max_slots=4096, streams=5, chunk=40, k=k)
    rng = np.random.default_rng(14)
    g, o = make_pair(w.capacity, w.max_slots, w.obs_bytes, w.act_bytes)
    add_both(g, o, rng, w.capacity)
    n_steps, per_round = 24, 6
    pipe = apex.Pipeline(g, depth, nb, w.k)
    rnd = rng.integers(0, U64, (n_steps, nb * w.k), dtype=np.uint64)
    newp = rng.lognormal(0, 1, (n_steps, nb * w.k)).astype(F32)
    d_rnd, d_newp = dev(rnd), dev(newp)
    S, T = w.streams, w.chunk
    scratch = [torch.empty(S * T, dtype=torch.float32, device="cuda:0") for _ in range(3)]
    rounds = []
    for i in range(n_steps // per_round):
        d = synth.actor_round(w, i)
        d["obs"] = rng.integers(0, 256, (S * T, w.obs_bytes), dtype=np.uint8)
        rounds.append((d, {k2: dev(v) for k2, v in d.items()}))
    torch.cuda.synchronize()
    assert pipe.fork() == 0
    refs, got = [], []
    for s in range(n_steps):
        if s % per_round == 0:
            d, dd = rounds[s // per_round]
            assert pipe.add_begin(dd["q_online"], dd["q_target"], dd["action"], dd["reward"], dd["discount"], w.n,
                                  dd["obs"], dd["act"], *scratch) == 0
        rc, first = pipe.steps(1, 0.4, d_rnd[s], d_newp[s])
        assert rc == 0 and first == s % depth
        rco, oo = o.sample(nb, w.k, 0.4, rnd[s])
        o.update_priorities(oo["key"], newp[s])
        refs.append(oo)
        if (s + 1) % per_round == 0:
            evict = (s + 1) % (2 * per_round) == 0
            rc, first_key, ev = pipe.add_end(evict)
            ref = oracle.nstep_priorities(d["q_online"], d["q_target"], d["action"], d["reward"], d["discount"],
                                          w.n, w.alpha, w.eps, w.frac_bits, w.max_slots)
            rco, fo = o.add(ref[0].reshape(-1), d["obs"], d["act"], ref[1].reshape(-1), ref[2].reshape(-1))
            assert (rc, first_key) == (rco, fo)
            if evict:
                assert o.evict() == (0, ev)
        # a set must be consumed before `depth` further steps are issued: copy it out now
        assert pipe.join() == 0
        torch.cuda.synchronize()
        got.append({k2: v.clone() for k2, v in pipe.sets[s % depth].items()})
        assert pipe.fork() == 0
    assert pipe.join() == 0
    torch.cuda.synchronize()
    for out, oo in zip(got, refs):
        assert_sample_equal(out, oo)
    check_gpu_tree(g, o)
    # several steps in one call, no synchronisation in between; the last `depth` sets are checked
    rnd2 = rng.integers(0, U64, (7, nb * w.k), dtype=np.uint64)
    newp2 = rng.lognormal(0, 1, (7, nb * w.k)).astype(F32)
    d2 = (dev(rnd2), dev(newp2))
    torch.cuda.synchronize()
    assert pipe.fork() == 0
    rc, first = pipe.steps(7, 0.4, *d2)
    assert rc == 0 and first == n_steps % depth
    assert pipe.join() == 0
    torch.cuda.synchronize()
    refs2 = []
    for s in range(7):
        rco, oo = o.sample(nb, w.k, 0.4, rnd2[s])
        o.update_priorities(oo["key"], newp2[s])
        refs2.append(oo)
    for s in range(7 - depth, 7):
        assert_sample_equal(pipe.sets[(n_steps + s) % depth], refs2[s])
    check_gpu_tree(g, o)
    pipe.close()


@pytest.mark.parametrize("nb,k", [(1, 64), (16, 128)])      # steps of one launch, steps with gathers on the copy streams
@pytest.mark.parametrize("second_fork", [None, "same", "other"])
def test_fork_and_join_order_the_copy_streams(nb, k, second_fork):
    """The copy streams are only asked to wait where they have to be: what a caller's stream writes late before a fork is
    seen by a payload copy of a later call, a further fork on the same stream or another one notwithstanding, and a stream
    that is joined sees the payload of a round that is still open and the rows that the copy streams gather."""
    from paper_1803_00933_amd import apex
    rng = np.random.default_rng(nb)
    T, ob, P = 240, 28224, 4000                     # 6.8 MB of observations: a round on the copy stream
    g, o = make_pair(P, P, ob, 4)
    assert add_both(g, o, rng, 2000) == 0
    pipe = apex.Pipeline(g, 3, nb, k)
    a, b, c = (torch.cuda.Stream() for _ in range(3))
    L = T + 1
    q = torch.zeros((1, L, 2), device="cuda:0")
    small = [torch.ones((1, L), device="cuda:0") for _ in range(2)]
    action = torch.zeros((1, L), dtype=torch.int32, device="cuda:0")
    act = torch.zeros((T, 4), dtype=torch.uint8, device="cuda:0")
    scratch = [torch.empty(T, device="cuda:0") for _ in range(3)]
    real = dev(rng.integers(0, 256, (T, ob), dtype=np.uint8))
    rnd, newp = dev(rng.integers(0, U64, (3, nb * k), dtype=np.uint64)), torch.ones((3, nb * k), device="cuda:0")
    for it in range(3):
        obs = torch.zeros((T, ob), dtype=torch.uint8, device="cuda:0")
        ring = g.obs_view()[2000 + it * T:2000 + (it + 1) * T]
        torch.cuda.synchronize()
        with torch.cuda.stream(a):
            torch.cuda._sleep(20_000_000)           # some ms
            obs.copy_(real)
        assert pipe.fork(a) == 0
        if second_fork:
            assert pipe.fork(a if second_fork == "same" else b) == 0
        assert pipe.add_begin(q, q, action, *small, 1, obs, act, *scratch) == 0
        assert pipe.steps(3, 0.4, rnd, newp)[0] == 0
        assert pipe.join(c) == 0
        with torch.cuda.stream(c):
            seen = [ring.clone()] + [s["obs"].clone() for s in pipe.sets]
        c.synchronize()
        torch.cuda.synchronize()
        assert torch.equal(seen[0], real)
        assert all(torch.equal(x, s["obs"]) for x, s in zip(seen[1:], pipe.sets))
        assert pipe.add_end()[0] == 0
        assert pipe.join(c) == 0
        torch.cuda.synchronize()
    pipe.close()


@pytest.mark.parametrize("streams", [48, 30])      # a round on the copy stream (5 MB), one on the learner's stream
def test_wide_steps_are_gathered_before_their_slots_are_reused(streams):
    """A ring with no slack: every add round lands in the slots that the eviction before it has just freed, and
    the batches drawn before that eviction hold many of the evicted keys.  Their gathers, which run on the copy
    streams, have to be through before the round's payload is written; nothing here synchronises in between."""
    from paper_1803_00933_amd import apex, synth
    nb, k, ob, depth, T = 4, 512, 4224, 4, 25
    count = streams * T
    C = 2100
    w = synth.WORKLOADS["tiny"].scaled(obs_bytes=ob, capacity=C, max_slots=C + count, streams=streams, chunk=T, k=k)
    rng = np.random.default_rng(streams)
    g, o = make_pair(w.capacity, w.max_slots, w.obs_bytes, w.act_bytes)
    add_both(g, o, rng, w.capacity)
    pipe = apex.Pipeline(g, depth, nb, w.k)
    cycles = 3 * depth
    rnd = rng.integers(0, U64, (cycles, nb * w.k), dtype=np.uint64)
    newp = rng.lognormal(0, 1, (cycles, nb * w.k)).astype(F32)
    d_rnd, d_newp = dev(rnd), dev(newp)
    scratch = [torch.empty(count, dtype=torch.float32, device="cuda:0") for _ in range(3)]
    rounds = []
    for i in range(cycles):
        d = synth.actor_round(w, i)
        d["obs"] = rng.integers(0, 256, (count, w.obs_bytes), dtype=np.uint8)
        rounds.append((d, {k2: dev(v) for k2, v in d.items()}))
    torch.cuda.synchronize()
    for c0 in range(0, cycles, depth):
        assert pipe.fork() == 0
        refs = []
        for s in range(c0, c0 + depth):
            d, dd = rounds[s]
            assert pipe.add_begin(dd["q_online"], dd["q_target"], dd["action"], dd["reward"], dd["discount"], w.n,
                                  dd["obs"], dd["act"], *scratch) == 0
            rc, first = pipe.steps(1, 0.4, d_rnd[s], d_newp[s])
            assert rc == 0 and first == s % depth
            rc, first_key, ev = pipe.add_end(True)
            refs.append(o.sample(nb, w.k, 0.4, rnd[s])[1])
            o.update_priorities(refs[-1]["key"], newp[s])
            ref = oracle.nstep_priorities(d["q_online"], d["q_target"], d["action"], d["reward"], d["discount"],
                                          w.n, w.alpha, w.eps, w.frac_bits, w.max_slots)
            assert (rc, first_key) == o.add(ref[0].reshape(-1), d["obs"], d["act"], ref[1].reshape(-1),
                                            ref[2].reshape(-1))
            assert o.evict() == (0, ev) and ev == count
        assert pipe.join() == 0
        torch.cuda.synchronize()
        for s in range(c0, c0 + depth):
            assert_sample_equal(pipe.sets[s % depth], refs[s - c0])
        check_gpu_tree(g, o)
    pipe.close()


def test_pipeline_small_and_large_add_rounds():
    """Small add rounds travel on the learner's stream, large ones on the copy stream: rounds of both kinds
    in one pipeline, with learner steps in between, against the oracle."""
    from paper_1803_00933_amd import apex, synth
    small = synth.WORKLOADS["tiny"].scaled(obs_bytes=4224, capacity=9000, max_slots=12288, streams=4, chunk=25, k=64)
    large = small.scaled(streams=40)              # 1000 rows of 4224 B: above the size that stays on one stream
    rng = np.random.default_rng(21)
    g, o = make_pair(small.capacity, small.max_slots, small.obs_bytes, small.act_bytes)
    add_both(g, o, rng, 8000)
    depth = 4
    pipe = apex.Pipeline(g, depth, 1, small.k)
    assert pipe.fork() == 0
    for i, w in enumerate([small, large, large, small, small, large, small]):
        d = synth.actor_round(w, i)
        n_rows = w.streams * w.chunk
        d["obs"] = rng.integers(0, 256, (n_rows, w.obs_bytes), dtype=np.uint8)
        dd = {k2: dev(v) for k2, v in d.items()}
        scratch = [torch.empty(n_rows, dtype=torch.float32, device="cuda:0") for _ in range(3)]
        rnd = rng.integers(0, U64, (3, w.k), dtype=np.uint64)
        newp = rng.lognormal(0, 1, (3, w.k)).astype(F32)
        d_rnd, d_newp = dev(rnd), dev(newp)
        assert pipe.add_begin(dd["q_online"], dd["q_target"], dd["action"], dd["reward"], dd["discount"], w.n,
                              dd["obs"], dd["act"], *scratch) == 0
        rc, first = pipe.steps(3, 0.4, d_rnd, d_newp)
        assert rc == 0
        rc, first_key, ev = pipe.add_end(True)
        refs = []
        for s in range(3):
            refs.append(o.sample(1, w.k, 0.4, rnd[s])[1])
            o.update_priorities(refs[-1]["key"], newp[s])
        ref = oracle.nstep_priorities(d["q_online"], d["q_target"], d["action"], d["reward"], d["discount"],
                                      w.n, w.alpha, w.eps, w.frac_bits, w.max_slots)
        rco, fo = o.add(ref[0].reshape(-1), d["obs"], d["act"], ref[1].reshape(-1), ref[2].reshape(-1))
        assert (rc, first_key) == (rco, fo)
        assert o.evict() == (0, ev)
        assert pipe.join() == 0
        torch.cuda.synchronize()
        for s in range(3):
            assert_sample_equal(pipe.sets[(first + s) % depth], refs[s])
        check_gpu_tree(g, o)
        assert pipe.fork() == 0
    assert pipe.join() == 0
    # the payload of the last rounds is where the oracle has it
    oo = sample_both(g, o, rng, 1, 64)
    pipe.close()


@pytest.mark.parametrize("ob", [256, 100, 7])
def test_small_add_round_rides_in_the_last_step_launch(ob):
    """With a small add round open (rows of at most 1 KB), the last step launch of a steps call is held back
    and issued by add_end with the round inside it; any other call issues it on its own.  Every order of
    calls against the oracle's plain order: steps, then the round, then the eviction."""
    from paper_1803_00933_amd import apex, synth
    w = synth.WORKLOADS["tiny"].scaled(obs_bytes=ob, capacity=9000, max_slots=12288, streams=6, chunk=25, k=96)
    rng = np.random.default_rng(ob)
    g, o = make_pair(w.capacity, w.max_slots, w.obs_bytes, w.act_bytes)
    add_both(g, o, rng, 8000)
    depth = 5
    pipe = apex.Pipeline(g, depth, 1, w.k)
    n_rows = w.streams * w.chunk
    scratch = [torch.empty(n_rows, dtype=torch.float32, device="cuda:0") for _ in range(3)]
    # (steps calls between add_begin and add_end, write-back, join before add_end, misaligned source rows)
    patterns = [([2], True, False, False), ([1, 1], True, False, False), ([1], True, True, False),
                ([], True, False, False), ([3], True, False, True), ([2], False, False, False),
                ([2], True, False, False)]
    assert pipe.fork() == 0
    for i, (calls, wb, join_between, misaligned) in enumerate(patterns):
        d = synth.actor_round(w, i)
        d["obs"] = rng.integers(0, 256, (n_rows, w.obs_bytes), dtype=np.uint8)
        dd = {k2: dev(v) for k2, v in d.items()}
        if misaligned:   # the same bytes at an address that is no multiple of 16 (nor of 4)
            buf = torch.empty(n_rows * ob + 64, dtype=torch.uint8, device="cuda:0")
            view = buf[3:3 + n_rows * ob].view(n_rows, ob)
            view.copy_(dd["obs"])
            dd["obs"] = view
        total = sum(calls)
        rnd = rng.integers(0, U64, (max(total, 1), w.k), dtype=np.uint64)
        newp = rng.lognormal(0, 1, (max(total, 1), w.k)).astype(F32)
        d_rnd, d_newp = dev(rnd), dev(newp)
        assert pipe.add_begin(dd["q_online"], dd["q_target"], dd["action"], dd["reward"], dd["discount"], w.n,
                              dd["obs"], dd["act"], *scratch) == 0
        firsts, at = [], 0
        for c in calls:
            rc, first = pipe.steps(c, 0.4, d_rnd[at:at + c], d_newp[at:at + c] if wb else None)
            assert rc == 0
            firsts += [(first + j) % depth for j in range(c)]
            at += c
        if join_between:
            assert pipe.join() == 0
            assert pipe.fork() == 0
        rc, first_key, ev = pipe.add_end(True)
        refs = []
        for s_ in range(total):
            refs.append(o.sample(1, w.k, 0.4, rnd[s_])[1])
            if wb:
                o.update_priorities(refs[-1]["key"], newp[s_])
        ref = oracle.nstep_priorities(d["q_online"], d["q_target"], d["action"], d["reward"], d["discount"],
                                      w.n, w.alpha, w.eps, w.frac_bits, w.max_slots)
        rco, fo = o.add(ref[0].reshape(-1), d["obs"], d["act"], ref[1].reshape(-1), ref[2].reshape(-1))
        assert (rc, first_key) == (rco, fo)
        assert o.evict() == (0, ev)
        assert pipe.join() == 0
        torch.cuda.synchronize()
        for s_ in range(total):
            assert_sample_equal(pipe.sets[firsts[s_]], refs[s_])
        check_gpu_tree(g, o)
        sample_both(g, o, rng, 2, 200)      # payload of the rounds added so far
        assert pipe.fork() == 0
    assert pipe.join() == 0
    st = g.stats()
    assert (st["size"], st["n_clamped"], st["n_stale_dropped"]) == (o.size, o.n_clamped, o.n_stale)
    pipe.close()


@pytest.mark.parametrize("ob,seed", [(64, 1), (64, 2), (4224, 3), (1040, 4), (100, 5), (256, 6), (28224, 7), (7, 8)])
def test_pipeline_random_call_orders(ob, seed):
    """Random orders of the pipeline's calls (steps of random length with and without write-back, add rounds
    opened and closed around them, evictions, joins, plain calls on the joined stream in between) against the
    oracle applying the same operations in the order of the calls."""
    from paper_1803_00933_amd import apex, synth
    rng = np.random.default_rng(seed)
    w = synth.WORKLOADS["tiny"].scaled(obs_bytes=ob, capacity=6000, max_slots=8192, streams=5, chunk=20, k=int(rng.integers(40, 130)))
    g, o = make_pair(w.capacity, w.max_slots, w.obs_bytes, w.act_bytes)
    add_both(g, o, rng, 5000)
    depth = int(rng.integers(3, 7))
    pipe = apex.Pipeline(g, depth, 1, w.k)
    n_rows = w.streams * w.chunk
    scratch = [torch.empty(n_rows, dtype=torch.float32, device="cuda:0") for _ in range(3)]
    keep = []               # device inputs stay alive until the next join
    pending = []            # (buffer set, oracle batch) to compare at the next join
    open_round = None
    assert pipe.fork() == 0
    for it in range(120):
        op = rng.choice(["steps", "steps", "steps", "begin", "end", "join", "plain"])
        if op == "steps":
            n = int(rng.integers(1, depth))          # fewer than the sets, so no set is overwritten before the join
            if len(pending) + n > depth:
                op = "join"
            else:
                wb = rng.random() < 0.8
                rnd = rng.integers(0, U64, (n, w.k), dtype=np.uint64)
                newp = rng.lognormal(0, 1.5, (n, w.k)).astype(F32)
                d_rnd, d_newp = dev(rnd), dev(newp)
                keep += [d_rnd, d_newp]
                rc, first = pipe.steps(n, 0.4, d_rnd, d_newp if wb else None)
                assert rc == 0
                for i in range(n):
                    rco, oo = o.sample(1, w.k, 0.4, rnd[i])
                    assert rco == 0
                    if wb:
                        assert o.update_priorities(oo["key"], newp[i]) == 0
                    pending.append(((first + i) % depth, oo))
        if op == "begin" and open_round is None and o.size + n_rows <= w.max_slots:
            d = synth.actor_round(w, it)
            d["obs"] = rng.integers(0, 256, (n_rows, w.obs_bytes), dtype=np.uint8)
            dd = {k2: dev(v) for k2, v in d.items()}
            keep.append(dd)
            assert pipe.add_begin(dd["q_online"], dd["q_target"], dd["action"], dd["reward"], dd["discount"], w.n,
                                  dd["obs"], dd["act"], *scratch) == 0
            open_round = d
        elif op == "end" and open_round is not None:
            d, open_round = open_round, None
            evict = bool(rng.random() < 0.5)
            rc, first_key, ev = pipe.add_end(evict)
            ref = oracle.nstep_priorities(d["q_online"], d["q_target"], d["action"], d["reward"], d["discount"],
                                          w.n, w.alpha, w.eps, w.frac_bits, w.max_slots)
            rco, fo = o.add(ref[0].reshape(-1), d["obs"], d["act"], ref[1].reshape(-1), ref[2].reshape(-1))
            assert (rc, first_key) == (rco, fo)
            if evict:
                assert o.evict() == (0, ev)
        elif op in ("join", "plain") and open_round is None:
            assert pipe.join() == 0
            torch.cuda.synchronize()
            for set_index, oo in pending:
                assert_sample_equal(pipe.sets[set_index], oo)
            pending, keep = [], []
            check_gpu_tree(g, o)
            if op == "plain":          # calls outside the pipeline change the first tree copy only
                oo = sample_both(g, o, rng, 1, 48)
                pr = rng.lognormal(0, 1, len(oo["key"])).astype(F32)
                assert g.update_priorities(dev(oo["key"]), dev(pr)) == o.update_priorities(oo["key"], pr) == 0
                if rng.random() < 0.3:
                    assert g.evict() == o.evict()
            assert pipe.fork() == 0
    if open_round is not None:
        rc, first_key, ev = pipe.add_end(False)
        d = open_round
        ref = oracle.nstep_priorities(d["q_online"], d["q_target"], d["action"], d["reward"], d["discount"],
                                      w.n, w.alpha, w.eps, w.frac_bits, w.max_slots)
        assert (rc, first_key) == o.add(ref[0].reshape(-1), d["obs"], d["act"], ref[1].reshape(-1), ref[2].reshape(-1))
    assert pipe.join() == 0
    torch.cuda.synchronize()
    for set_index, oo in pending:
        assert_sample_equal(pipe.sets[set_index], oo)
    check_gpu_tree(g, o)
    st = g.stats()
    assert (st["size"], st["n_clamped"], st["n_stale_dropped"]) == (o.size, o.n_clamped, o.n_stale)
    pipe.close()


@pytest.mark.parametrize("nb,k,ob", PIPELINE_STEP_SHAPES)
def test_pipeline_graph_replays(nb, k, ob):
    """One cycle (an add round beside six learner steps, then eviction) captured as a HIP graph by the
    pipeline and replayed; every replay is checked against the oracle, with eager work in between."""
    from paper_1803_00933_amd import apex, synth
    w = synth.WORKLOADS["tiny"].scaled(obs_bytes=ob, capacity=3000, max_slots=4096, streams=5, chunk=40, k=k)
    rng = np.random.default_rng(15)
    g, o = make_pair(w.capacity, w.max_slots, w.obs_bytes, w.act_bytes)
    add_both(g, o, rng, w.capacity)
    depth, n_steps = 3, 6
    pipe = apex.Pipeline(g, depth, nb, w.k)
    rnd = rng.integers(0, U64, (n_steps, nb * w.k), dtype=np.uint64)
    newp = rng.lognormal(0, 1, (n_steps, nb * w.k)).astype(F32)
    d_rnd, d_newp = dev(rnd), dev(newp)
    S, T = w.streams, w.chunk
    scratch = [torch.empty(S * T, dtype=torch.float32, device="cuda:0") for _ in range(3)]
    d = synth.actor_round(w, 0)
    d["obs"] = rng.integers(0, 256, (S * T, w.obs_bytes), dtype=np.uint8)
    dd = {k2: dev(v) for k2, v in d.items()}
    torch.cuda.synchronize()

    def cycle():
        assert pipe.add_begin(dd["q_online"], dd["q_target"], dd["action"], dd["reward"], dd["discount"], w.n,
                              dd["obs"], dd["act"], *scratch) == 0
        assert pipe.steps(n_steps, 0.4, d_rnd, d_newp)[0] == 0
        rc, _, ev = pipe.add_end(True)
        assert (rc, ev) == (0, S * T)

    def oracle_cycle():
        res = []
        for s in range(n_steps):
            res.append(o.sample(nb, w.k, 0.4, rnd[s])[1])
            o.update_priorities(res[-1]["key"], newp[s])
        ref = oracle.nstep_priorities(d["q_online"], d["q_target"], d["action"], d["reward"], d["discount"],
                                      w.n, w.alpha, w.eps, w.frac_bits, w.max_slots)
        assert o.add(ref[0].reshape(-1), d["obs"], d["act"], ref[1].reshape(-1), ref[2].reshape(-1))[0] == 0
        assert o.evict() == (0, S * T)
        return res

    assert pipe.capture_begin() == 0
    cycle()
    assert pipe.capture_end() == 0
    for replay in range(4):
        assert pipe.fork() == 0
        assert pipe.replay(1) == 0
        assert pipe.join() == 0
        torch.cuda.synchronize()
        res = oracle_cycle()
        for s in range(n_steps - depth, n_steps):
            assert_sample_equal(pipe.sets[s % depth], res[s])
        assert g.resync() == 0
        check_gpu_tree(g, o)
        if replay == 1:                       # eager calls between replays, on the same memory
            add_both(g, o, rng, 30)
            sample_both(g, o, rng, 1, 32)
            assert g.evict() == o.evict()
    # several replays back to back
    assert pipe.fork() == 0
    assert pipe.replay(3) == 0
    assert pipe.join() == 0
    torch.cuda.synchronize()
    for _ in range(3):
        res = oracle_cycle()
    for s in range(n_steps - depth, n_steps):
        assert_sample_equal(pipe.sets[s % depth], res[s])
    assert g.resync() == 0
    check_gpu_tree(g, o)
    pipe.close()


@pytest.mark.parametrize("P,C,k,ob", [
    (4096, 3000, 96, 4224),          # one tree level
    (40_000, 30_000, 200, 4112),     # two levels, ragged tails, partial last vector chunk
    (400_000, 300_000, 512, 4224),   # three levels
    (5000, 4000, 1024, 32768),       # as many samples as a workgroup has lanes, largest fused row
    (5000, 4000, 1, 4224),           # batches of one
    (60_000, 50_000, 512, 256),      # short rows (feature vectors): a few lanes of each workgroup copy
    (70_000, 60_000, 300, 4224),     # a summit of 274 nodes over 1094
    (280_000, 250_000, 256, 1040),   # a summit of 274 nodes over 4375, a ragged one
    (4608, 4000, 64, 4112),          # a summit over the leaves
    (33_000, 30_000, 517, 2064),     # 516 top nodes (two reads of the drawing wave), k no multiple of 8
    (65_536, 60_000, 128, 4112),     # 1024 top nodes, the most without a summit
    (1000, 900, 64, 64),             # 1000 top nodes that are the leaves
    (9000, 8000, 1000, 48),          # two passes over the pending pairs, a ragged last one
    (5000, 4000, 100, 4100),         # rows that are no multiple of 16 bytes: the last piece overlaps the one before
    (3000, 2500, 64, 1001),          # odd row size: unaligned pieces
    (3000, 2500, 96, 56448),         # rows longer than one pass of a workgroup (two frame stacks per transition)
    (3000, 2500, 40, 32784),         # just beyond one pass
])
def test_one_launch_per_learner_step(P, C, k, ob):
    """Sequences of learner steps issued as one launch per step (draw of the next batch inside the launch
    that gathers and writes back the current one, two copies of the tree): every batch of every sequence
    against the oracle doing draw, update, draw, update, with other operations between the sequences.
    Priorities are heavy-tailed so that batches draw the same slot several times."""
    from paper_1803_00933_amd import apex
    rng = np.random.default_rng(P + k)
    g, o = make_pair(C, P, ob, 4)
    heavy = lambda rng, n: (rng.pareto(0.4, n) + 1e-3)
    while o.size < C:
        assert add_both(g, o, rng, min(20_000, C - o.size), heavy) == 0
    depth = 9
    pipe = apex.Pipeline(g, depth, 1, k)
    for seq in range(6):
        n = (8, 2, 8, 8, 1, 7)[seq]           # sequences of one and two steps never read the second tree copy
        rnd = rng.integers(0, U64, (n, k), dtype=np.uint64)
        newp = heavy(rng, (n, k)).astype(F32)
        newp[rng.random((n, k)) < 0.1] = 0.0
        with_update = seq != 3
        d_rnd, d_newp = dev(rnd), dev(newp)
        torch.cuda.synchronize()
        assert pipe.fork() == 0
        rc, first = pipe.steps(n, 0.5, d_rnd, d_newp if with_update else None)
        assert rc == 0
        assert pipe.join() == 0
        torch.cuda.synchronize()
        dup = 0
        for i in range(n):
            rco, oo = o.sample(1, k, 0.5, rnd[i])
            assert rco == 0
            dup += k - len(np.unique(oo["slot"]))
            if with_update:
                assert o.update_priorities(oo["key"], newp[i]) == 0
            assert_sample_equal(pipe.sets[(first + i) % depth], oo)
        assert k < 64 or n < 7 or dup > 0  # the case the test is about occurs
        check_gpu_tree(g, o)
        # other operations between the sequences: they change the first copy of the tree only
        if seq % 2 == 0:
            assert add_both(g, o, rng, min(500, P - o.size), heavy) == 0
            assert g.evict() == o.evict()
        else:
            oo = sample_both(g, o, rng, 1, min(k, 64))
            pr = heavy(rng, len(oo["key"])).astype(F32)
            assert g.update_priorities(dev(oo["key"]), dev(pr)) == o.update_priorities(oo["key"], pr) == 0
    st = g.stats()
    assert (st["n_clamped"], st["n_stale_dropped"]) == (o.n_clamped, o.n_stale)
    pipe.close()


@pytest.mark.parametrize("ob", [1024, 1025, 1028, 4096, 4097])
@pytest.mark.parametrize("nb,k", [(1, 1024), (2, 512), (5, 33), (2, 513)])
def test_steps_that_are_no_single_launch(ob, nb, k):
    """Pipeline steps of two buffer sets or several batches, rows and batches on both sides of the lines between the
    write-back spread over the copying workgroups and an update of its own, and the same through the plain halves.
    Heavy-tailed priorities: batches draw slots several times."""
    from paper_1803_00933_amd import apex
    rng = np.random.default_rng(ob + k)
    g, o = make_pair(3000, 3500, ob, 4)
    heavy = lambda rng, n: rng.pareto(0.4, n) + 1e-3
    assert add_both(g, o, rng, 3000, heavy) == 0
    n, per = 3, nb * k
    pipe = apex.Pipeline(g, 2, nb, k)
    rnd, newp = rng.integers(0, U64, (n, per), dtype=np.uint64), heavy(rng, (n, per)).astype(F32)
    d_rnd, d_newp = dev(rnd), dev(newp)
    assert pipe.fork() == 0 and pipe.steps(n, 0.4, d_rnd, d_newp)[0] == 0 and pipe.join() == 0
    torch.cuda.synchronize()
    for i in range(n):
        oo = o.sample(nb, k, 0.4, rnd[i])[1]
        assert len(np.unique(oo["slot"])) < per
        assert o.update_priorities(oo["key"], newp[i]) == 0
        if i >= n - 2:
            assert_sample_equal(pipe.sets[i % 2], oo)
    check_gpu_tree(g, o)
    out = g.alloc_sample_outputs(nb, k)
    out["mass"] = torch.empty(per, dtype=torch.int64, device="cuda:0")
    oo = o.sample(nb, k, 0.4, rnd[0])[1]
    assert o.update_priorities(oo["key"], newp[1]) == 0
    assert g.sample_begin(nb, k, d_rnd[0], out) == 0
    assert g.sample_finish_writeback(nb, k, 0.4, out, d_newp[1]) == 0
    torch.cuda.synchronize()
    assert_sample_equal(out, oo)
    check_gpu_tree(g, o)
    pipe.close()


@pytest.mark.parametrize("P,ob,nb,k,depth,bits", [
    (900, 16, 33, 3, 2, 24), (900, 20, 17, 50, 3, 24), (3000, 64, 16, 65, 4, 24), (3000, 7, 100, 2, 2, 24),   # batches per row
    (40_000, 100, 2, 1100, 2, 24), (70_000, 12, 40, 40, 3, 24), (5000, 300, 1, 1025, 3, 24),   # wide top, summit, one batch
    (30, 16, 5, 64, 2, 0), (30, 16, 20, 17, 3, 1), (4000, 4096, 3, 16, 5, 24),                 # no mass for a stratum
])
def test_steps_of_several_batches_in_one_launch_each(P, ob, nb, k, depth, bits):
    """Sequences of steps of several batches (or of one large one) against the oracle: batches that draw one another's
    slots again and again (which of them is the last is told from the uniforms), strata smaller than a mass and of no
    width at all, calls of one and of several steps, add rounds, evictions, plain updates and steps without write-back in
    between, and replays of a captured sequence."""
    from paper_1803_00933_amd import apex
    rng = np.random.default_rng(P + nb * k)
    C = P - P // 10
    g, o = make_pair(C, P, ob, 4, frac_bits=bits)
    heavy = lambda rng, n: np.where(rng.random(n) < 0.2, 0.0, rng.pareto(0.5, n) + 1e-3)
    assert add_both(g, o, rng, C, heavy) == 0
    pipe, per, at = apex.Pipeline(g, depth, nb, k), nb * k, 0

    def steps(n, write_back=True):
        nonlocal at
        rnd, newp = rng.integers(0, U64, (n, per), dtype=np.uint64), heavy(rng, (n, per)).astype(F32)
        rnd[0, ::5], rnd[0, 1::5] = 0, U64 - 1
        newp[rng.random((n, per)) < 0.05] = np.inf
        args = dev(rnd), dev(newp) if write_back else None
        torch.cuda.synchronize()
        assert pipe.fork() == 0
        assert pipe.steps(n, 0.4, *args) == (0, at % depth)
        assert pipe.join() == 0
        torch.cuda.synchronize()
        for i in range(n):
            rco, oo = o.sample(nb, k, 0.4, rnd[i])
            assert rco == 0
            if write_back:
                assert o.update_priorities(oo["key"], newp[i]) == 0
            if i >= n - depth:
                assert_sample_equal(pipe.sets[(at + i) % depth], oo)
        at += n
        return check_gpu_tree(g, o)

    for it in range(4):
        steps(3)
        steps(1)
        assert add_both(g, o, rng, P // 20, heavy) == 0
        steps(2)
        assert g.evict() == o.evict()
        steps(1)
        oo = sample_both(g, o, rng, 1, 40)
        pr = rng.lognormal(0, 1, 40).astype(F32)
        assert g.update_priorities(dev(oo["key"]), dev(pr)) == o.update_priorities(oo["key"], pr) == 0
        steps(1 if it % 2 else 2)
        steps(2, write_back=False)
    rnd, newp = rng.integers(0, U64, (2, per), dtype=np.uint64), heavy(rng, (2, per)).astype(F32)
    args = dev(rnd), dev(newp)
    torch.cuda.synchronize()
    assert pipe.capture_begin() == 0
    assert pipe.steps(2, 0.4, *args)[0] == 0
    assert pipe.capture_end() == 0
    first = at
    at += 2
    for it in range(3):
        assert pipe.replay() == 0 and pipe.join() == 0
        torch.cuda.synchronize()
        for i in range(2):
            rco, oo = o.sample(nb, k, 0.4, rnd[i])
            assert rco == 0 and o.update_priorities(oo["key"], newp[i]) == 0
            assert_sample_equal(pipe.sets[(first + i) % depth], oo)
        check_gpu_tree(g, o)
        oo = sample_both(g, o, rng, 1, 33)
        assert g.update_priorities(dev(oo["key"]), dev(np.ones(33, F32))) == o.update_priorities(oo["key"], np.ones(33, F32)) == 0
    steps(3)
    pipe.close()


@pytest.mark.parametrize("ob,k,extra", [(28224, 512, 0), (4224, 100, 0), (64, 128, 0), (4224, 700, 600),
                                        (64, 700, 600), (7, 512, 700)])   # short rows, more than 1024 pairs
def test_finish_with_update_riding_along(ob, k, extra):
    """apex_replay_sample_finish_update == finish, then update (in the gather kernel's extra workgroup when
    the batch fits one; with short rows the first pass of a larger update rides in the gather launch; by
    launches of its own otherwise)."""
    rng = np.random.default_rng(16 + k)
    g, o = make_pair(3000, 4096, ob, 4)
    add_both(g, o, rng, 3000)
    for step in range(4):
        rnd = rng.integers(0, U64, k, dtype=np.uint64)
        rco, oo = o.sample(1, k, 0.4, rnd)
        keys = np.concatenate([oo["key"], rng.integers(0, 3000, extra).astype(np.uint64)])   # extra: > 1024 pairs
        newp = rng.lognormal(0, 1, len(keys)).astype(F32)
        o.update_priorities(keys, newp)
        out = g.alloc_sample_outputs(1, k)
        out["mass"] = torch.empty(k, dtype=torch.int64, device="cuda:0")
        assert g.sample_begin(1, k, dev(rnd), out) == 0
        assert g.sample_finish_update(1, k, 0.4, out, dev(keys), dev(newp)) == 0
        torch.cuda.synchronize()
        assert_sample_equal(out, oo)
        check_gpu_tree(g, o)
        # the batch's own priorities written back by the launch that finishes it
        rnd = rng.integers(0, U64, k, dtype=np.uint64)
        rco, oo = o.sample(1, k, 0.4, rnd)
        newp = rng.lognormal(0, 1, k).astype(F32)
        o.update_priorities(oo["key"], newp)
        assert g.sample_begin(1, k, dev(rnd), out) == 0
        assert g.sample_finish_writeback(1, k, 0.4, out, dev(newp)) == 0
        torch.cuda.synchronize()
        assert_sample_equal(out, oo)
        check_gpu_tree(g, o)
        # several batches per call: samples of different batches collide on heavy transitions
        nb = 3
        rnd = rng.integers(0, U64, nb * k, dtype=np.uint64)
        rco, oo = o.sample(nb, k, 0.4, rnd)
        newp = rng.lognormal(0, 1, nb * k).astype(F32)
        o.update_priorities(oo["key"], newp)
        out3 = g.alloc_sample_outputs(nb, k)
        out3["mass"] = torch.empty(nb * k, dtype=torch.int64, device="cuda:0")
        assert g.sample_begin(nb, k, dev(rnd), out3) == 0
        assert g.sample_finish_writeback(nb, k, 0.4, out3, dev(newp)) == 0
        torch.cuda.synchronize()
        assert_sample_equal(out3, oo)
        check_gpu_tree(g, o)


@pytest.mark.parametrize("ob,k,extra", [(16, 256, 900), (16, 257, 900), (33, 511, 700), (1024, 512, 600), (1000, 513, 600),
                                        (4096, 256, 800), (4096, 300, 800), (2049, 1025, 0)])
def test_finish_around_a_workgroup_of_weights(ob, k, extra):
    """Rows, weights and the first pass of an update in one launch: workgroups of 512 from 257 weights on, at their edges."""
    test_finish_with_update_riding_along(ob, k, extra)


@pytest.mark.parametrize("m,A", [(512, 18), (96, 1), (3000, 4)])
def test_update_from_learner_q_values(m, A):
    """apex_replay_update_from_q: priorities recomputed from the stored (ret, gacc) and fresh Q-values, in the
    one-workgroup path and in the two-pass path, with repeats and stale keys."""
    rng = np.random.default_rng(17 + m)
    g, o = make_pair(5000, 8192, 16, 4)
    add_both(g, o, rng, 5000)
    add_both(g, o, rng, 2000)
    assert g.evict() == o.evict()                      # keys 0..1999 are stale now
    for it in range(3):
        keys = rng.integers(1500, 7300, m).astype(np.uint64)      # some stale, some not yet added, many repeats
        q_taken = rng.standard_normal(m).astype(F32)
        q_on = np.round(rng.standard_normal((m, A)) * 2).astype(F32) / 2       # ties in the argmax
        q_tg = rng.standard_normal((m, A)).astype(F32)
        rco, p_ref = o.update_from_q(keys, q_taken, q_on, q_tg)
        p_out = torch.empty(m, dtype=torch.float32, device="cuda:0")
        rcg = g.update_from_q(dev(keys), dev(q_taken), dev(q_on), dev(q_tg), p_out)
        assert rcg == rco == 0
        torch.cuda.synchronize()
        assert np.array_equal(host(p_out).view(np.uint32), p_ref.view(np.uint32))
        check_gpu_tree(g, o)
    sample_both(g, o, rng, 2, 128)


@pytest.mark.parametrize("act_bytes", [1, 2, 3, 4, 5, 7, 15, 16, 17])
@pytest.mark.parametrize("obs_bytes,with_obs", [(4112, True), (64, False)])
def test_small_columns_of_a_whole_add(act_bytes, obs_bytes, with_obs):
    """The columns that a whole add brings along with the masses (up to 16 action bytes) or in a launch of their own,
    each of them possibly missing, on a ring that wraps: what is there lands in its rows, the rest stays."""
    from paper_1803_00933_amd import apex
    rng = np.random.default_rng(act_bytes)
    P, count = 2500, 1100  # more than one workgroup of transitions
    g = apex.Replay(1200, P, obs_bytes, act_bytes)
    for view in (g.obs_view(), g.act_view(), g.ret_view(), g.gacc_view()):
        view.zero_()
    want = [np.zeros((P, act_bytes), np.uint8), np.zeros(P, np.float32), np.zeros(P, np.float32)]
    obs = rng.integers(0, 256, (count, obs_bytes), dtype=np.uint8)
    for it in range(8):
        cols = [rng.integers(0, 256, (count, act_bytes), dtype=np.uint8), rng.standard_normal(count).astype(np.float32),
                rng.random(count).astype(np.float32)]
        given = [it & (1 << b) == 0 for b in range(3)]
        args = [dev(c) if there else None for c, there in zip(cols, given)]
        prio = rng.lognormal(0, 1, count).astype(np.float32)
        rc, first = g.add(dev(prio), dev(obs) if with_obs else None, *args)
        assert rc == 0 and first == it * count
        rows = (first + np.arange(count)) % P
        for w, c, there in zip(want, cols, given):
            if there:
                w[rows] = c
        torch.cuda.synchronize()
        assert np.array_equal(host(g.act_view(), np.uint8).reshape(P, act_bytes), want[0])
        assert np.array_equal(host(g.ret_view(), np.float32), want[1])
        assert np.array_equal(host(g.gacc_view(), np.float32), want[2])
        if with_obs:
            assert np.array_equal(host(g.obs_view(), np.uint8).reshape(P, obs_bytes)[rows], obs)
        assert g.evict()[0] == 0


# Shares of the weights (512 samples each), steps that add neighbouring changes up before they go to the upper levels and
# steps that do not, and both sides of the lines beyond which steps are two launches each: batches, samples per top node.
@pytest.mark.parametrize("P,ob,nb,k,depth", [
    (3000, 16, 1, 8192, 2), (70_000, 12, 1, 8191, 2), (200_000, 7, 3, 513, 3), (9000, 20, 2, 1025, 2),      # shares
    (20_000, 16, 3, 1001, 2), (300_000, 12, 8, 512, 2), (40_000, 8, 1, 8190, 2),                            # added up
    (300_000, 12, 16, 512, 2), (5000, 20, 160, 9, 2), (5000, 20, 161, 9, 2),                                # the lines
])
def test_steps_of_large_and_of_many_batches(P, ob, nb, k, depth):
    test_steps_of_several_batches_in_one_launch_each(P, ob, nb, k, depth, 24)


# replay.Sample on both sides of the lines beyond which long rows, and large batches of rows that do not all find room on the
# chip at once, are two launches; two and four pieces per lane on both sides of a full chip.
@pytest.mark.parametrize("ob,nb,k", [
    (98_304, 1, 40), (98_305, 1, 40), (98_320, 1, 33), (53_248, 1, 513), (53_249, 1, 513), (32_768, 1, 769), (32_769, 1, 769),
    (28_688, 1, 768), (28_688, 1, 769), (28_688, 3, 384), (28_688, 2, 385), (16_384, 1, 768), (16_384, 1, 769), (20_000, 1, 512),
    (20_001, 1, 513),
])
def test_samples_of_long_rows_at_the_edges_of_their_rule(ob, nb, k):
    rng = np.random.default_rng(ob + k)
    g, o = make_pair(700, 800, ob, 4)
    assert add_both(g, o, rng, 700) == 0
    for _ in range(2):
        sample_both(g, o, rng, nb, k)


@pytest.mark.parametrize("obs_bytes", [16, 7])
def test_the_largest_adds_of_short_rows(obs_bytes):
    """Adds of so many short rows that they go in the largest workgroups, over the end of the ring."""
    rng = np.random.default_rng(obs_bytes)
    P = 450_000
    g, o = make_pair(1000, P, obs_bytes, 4)
    for cnt in (200_000, 200_001, 300_333):
        obs, act = (rng.integers(0, 256, (cnt, n), dtype=np.uint8) for n in (obs_bytes, 4))
        ret, gacc, prio = rng.standard_normal(cnt).astype(F32), rng.random(cnt).astype(F32), rng.lognormal(0, 1, cnt).astype(F32)
        rc, first = g.add(dev(prio), dev(obs), dev(act), dev(ret), dev(gacc))
        assert (rc, first) == o.add(prio, obs, act, ret, gacc) and rc == 0
        rows = (first + np.arange(cnt)) % P
        torch.cuda.synchronize()
        assert np.array_equal(host(g.obs_view()).reshape(P, obs_bytes)[rows], obs)
        assert np.array_equal(host(g.act_view()).reshape(P, 4)[rows], act)
        assert np.array_equal(host(g.ret_view())[rows], ret) and np.array_equal(host(g.gacc_view())[rows], gacc)
        check_gpu_tree(g, o)
        assert g.evict() == o.evict()
    check_gpu_tree(g, o)


# Steps of several batches of short rows, and of one large one, take one launch each, which leaves both copies of the tree
# behind: add rounds in between, as one launch or from the copy stream, have to keep them alike.
SEVERAL_BATCH_SHAPES = [(3, 100, 64), (1, 1100, 256), (20, 33, 7)]


@pytest.mark.parametrize("depth", [3, 2])
@pytest.mark.parametrize("nb,k,ob", SEVERAL_BATCH_SHAPES)
def test_steps_of_several_batches_beside_add_rounds(nb, k, ob, depth):
    test_pipeline_matches_the_plain_call_order(nb, k, ob, depth)


@pytest.mark.parametrize("nb,k,ob", SEVERAL_BATCH_SHAPES)
def test_steps_of_several_batches_beside_add_rounds_replayed(nb, k, ob):
    test_pipeline_graph_replays(nb, k, ob)


@pytest.mark.parametrize("nb,k", [(3, 100), (1, 1100)])
def test_steps_of_several_batches_beside_small_and_large_add_rounds(nb, k):
    """Rounds below and above 4 MB of observations, the latter from the copy stream, with steps of several batches in
    between that read what the rounds have left in either copy of the tree."""
    from paper_1803_00933_amd import apex, synth
    small = synth.WORKLOADS["tiny"].scaled(obs_bytes=4096, capacity=9000, max_slots=12288, streams=4, chunk=25, k=k)
    large = small.scaled(streams=44)              # 1100 rows of 4096 B
    rng = np.random.default_rng(k)
    g, o = make_pair(small.capacity, small.max_slots, small.obs_bytes, small.act_bytes)
    add_both(g, o, rng, 8000)
    depth = 4
    pipe = apex.Pipeline(g, depth, nb, k)
    assert pipe.fork() == 0
    for i, w in enumerate([small, large, large, small, large, small]):
        d = synth.actor_round(w, i)
        n_rows = w.streams * w.chunk
        d["obs"] = rng.integers(0, 256, (n_rows, w.obs_bytes), dtype=np.uint8)
        dd = {k2: dev(v) for k2, v in d.items()}
        scratch = [torch.empty(n_rows, dtype=torch.float32, device="cuda:0") for _ in range(3)]
        rnd = rng.integers(0, U64, (4, nb * k), dtype=np.uint64)
        newp = rng.lognormal(0, 1, (4, nb * k)).astype(F32)
        d_rnd, d_newp = dev(rnd), dev(newp)
        torch.cuda.synchronize()
        assert pipe.add_begin(dd["q_online"], dd["q_target"], dd["action"], dd["reward"], dd["discount"], w.n,
                              dd["obs"], dd["act"], *scratch) == 0
        rc, first = pipe.steps(3, 0.4, d_rnd, d_newp)
        assert rc == 0
        rc, first_key, ev = pipe.add_end(i % 2 == 0)
        assert pipe.steps(1, 0.4, d_rnd[3], d_newp[3])[0] == 0
        refs = []
        for s in range(4):
            if s == 3:
                ref = oracle.nstep_priorities(d["q_online"], d["q_target"], d["action"], d["reward"], d["discount"],
                                              w.n, w.alpha, w.eps, w.frac_bits, w.max_slots)
                rco, fo = o.add(ref[0].reshape(-1), d["obs"], d["act"], ref[1].reshape(-1), ref[2].reshape(-1))
                assert (rc, first_key) == (rco, fo)
                if i % 2 == 0:
                    assert o.evict() == (0, ev)
            refs.append(o.sample(nb, k, 0.4, rnd[s])[1])
            o.update_priorities(refs[-1]["key"], newp[s])
        assert pipe.join() == 0
        torch.cuda.synchronize()
        for s in range(4):
            assert_sample_equal(pipe.sets[(first + s) % depth], refs[s])
        check_gpu_tree(g, o)
        assert pipe.fork() == 0
    assert pipe.join() == 0
    pipe.close()


# Batches around the edges of what a wave reads of the board together, of the odd word at a batch's end, of the lines between
# board and tickets (1024 samples, 128 per batch) and between the kernels; rows on both sides of the streaming stores.
@pytest.mark.parametrize("ob,ab,nb,k", [
    (16, 1, 1, 1), (16, 3, 1024, 1), (20, 4, 3, 2), (31, 5, 16, 63), (268, 84, 2, 65), (255, 4, 12, 100), (256, 4, 12, 100),
    (256, 255, 11, 128), (256, 256, 7, 129), (2047, 257, 8, 128), (2048, 300, 3, 500), (2048, 2, 2, 512), (1023, 4, 1, 768),
    (1023, 4, 1, 769), (1024, 4, 1, 1024), (4096, 4, 3, 341), (28224, 4, 3, 333), (33000, 4, 1, 129),
    (1024, 4, 1, 832), (2047, 4, 1, 833), (2048, 4, 1, 1024),
])
def test_weights_by_the_board(ob, ab, nb, k):
    """replay.Sample with a workgroup per sample: every weight, again and again and in replays of one captured call, with calls
    of other sizes and of the kernels that take tickets in between; the words of the board are 0 again afterwards, and words
    that overlapping calls have left there (planted) are gone two calls later."""
    rng = np.random.default_rng(ob + k)
    g, o = make_pair(1100, 1200, ob, ab)
    assert add_both(g, o, rng, 1100, lambda r, n: r.pareto(1.1, n)) == 0
    for n, m in ((nb, k), (1, 40), (nb, k), (nb, k), (2, 700), (nb, k)):
        sample_both(g, o, rng, n, m)
    rnd = rng.integers(0, U64, nb * k, dtype=np.uint64)
    out, d_rnd = g.alloc_sample_outputs(nb, k), dev(rnd)
    ref = o.sample(nb, k, 0.4, rnd)[1]
    s, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=s):
        assert g.sample(nb, k, 0.4, d_rnd, out=out)[0] == 0
    for _ in range(3):
        out["weight"].fill_(-1.0)
        graph.replay()
        torch.cuda.synchronize()
        assert_sample_equal(out, ref)
        sample_both(g, o, rng, 2, 33)
    board = g.scratch[-4 * 4 * 16384:].view(torch.int32)       # the last region: four sets of 4096 words, 16 of every 64
    torch.cuda.synchronize()
    assert int(board.abs().max()) == 0
    board.view(-1, 64)[:, :16] = 0x3f800000
    for _ in range(2):
        assert g.sample(nb, k, 0.4, d_rnd, out=out)[0] == 0
    for _ in range(4):
        sample_both(g, o, rng, nb, k)


@pytest.mark.parametrize("P", [512, 1024, 30_000, 300_000])
def test_carries_in_prefix_sums(P):
    """Masses whose low words carry in every step of a 64-bit prefix sum and in every lane, and masses of which only some do:
    draws by one wave alone, by a workgroup per sample and by 16 lanes, updates and add rounds, bit for bit."""
    rng = np.random.default_rng(P)
    carrying = F32(1 - 2.0 ** -20)                # a mass of 2^32 - 2^12, give or take some hundred
    some = lambda r, n: np.where(r.random(n) < 0.5, carrying, F32(2.0 ** -28))
    for dist in (lambda r, n: np.full(n, carrying), some):
        g, o = make_pair(P - 300, P, 16, 4, alpha=1.0, eps=0.0, frac_bits=32)
        assert add_both(g, o, rng, P - 300, dist) == 0
        assert int((o.leaves() & 0x80000000).max()) != 0
        check_gpu_tree(g, o)
        for nb, k in ((1, 1), (1, 300), (1, 1500), (3, 600), (1, 4096)):
            oo = sample_both(g, o, rng, nb, k)
            pr = some(rng, len(oo["key"])).astype(F32)
            assert g.update_priorities(dev(oo["key"]), dev(pr)) == o.update_priorities(oo["key"], pr) == 0
            check_gpu_tree(g, o)
        assert add_both(g, o, rng, 257, dist) == 0
        check_gpu_tree(g, o)
        sample_both(g, o, rng, 2, 64)
        assert g.evict() == o.evict()
        check_gpu_tree(g, o)
