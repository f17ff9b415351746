"""GPU parity: the memory with prioritized eviction (apex_pe_*) against its oracle."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import assert_sample_equal, dev, host

pytestmark = pytest.mark.gpu
F32 = np.float32
U64 = 1 << 64


def check(g, o):
    lay = g.layout
    for which in (False, True):
        levels = [host(g.level_view(l, which), np.uint64) for l in range(lay.tree_levels)]
        assert np.array_equal(levels[0], o.leaves(which)), "leaves %s" % which
        for l in range(1, lay.tree_levels):
            child = levels[l - 1]
            pad = (-len(child)) % lay.tree_fanout
            sums = np.concatenate([child, np.zeros(pad, np.uint64)]).reshape(-1, lay.tree_fanout).sum(1, dtype=np.uint64)
            assert np.array_equal(levels[l], sums), "level %d %s" % (l, which)
    st = g.stats()
    assert (st["root"], st["root_evict"]) == (o.root, o.root_evict)
    assert (st["size"], st["inserted"], st["evicted"]) == (o.size, o.inserted, o.evicted)
    assert (st["free_head"], st["free_tail"]) == (o.free_head, o.free_tail)
    assert (st["n_stale_dropped"], st["n_clamped"]) == (o.n_stale, o.n_clamped)
    assert np.array_equal(host(g.gen_view(), np.uint32), o.gen())
    P = o.max_slots
    idx = np.arange(o.free_head, o.free_tail) % P
    assert np.array_equal(host(g.free_ring_view(), np.uint32)[idx], o.free_ring()[idx])     # the live part of the ring


@pytest.mark.parametrize("P,C,ob,ab", [(600, 400, 32, 4), (70_000, 60_000, 4112, 8), (400_000, 300_000, 12, 4)])
def test_random_sequences_with_prioritized_eviction(P, C, ob, ab):
    from paper_1803_00933_amd import apex
    rng = np.random.default_rng(P)
    g = apex.PeReplay(C, P, ob, ab)
    o = oracle.PrioritizedEvictionReplay(C, P, ob, ab)
    rounds = 6
    for it in range(8):
        cnt = P - o.size if it == 0 else int(rng.integers(1, P - o.size + 1))
        obs = rng.integers(0, 256, (cnt, ob), dtype=np.uint8)
        act = rng.integers(0, 256, (cnt, ab), dtype=np.uint8)
        ret, gacc = rng.standard_normal(cnt).astype(F32), rng.random(cnt).astype(F32)
        prio = np.where(rng.random(cnt) < 0.1, 0.0, rng.lognormal(0, 1.5, cnt)).astype(F32)
        assert o.add(prio, obs, act, ret, gacc)[0] == 0
        assert g.add(dev(prio), dev(obs), dev(act), dev(ret), dev(gacc)) == 0
        assert g.add(dev(np.ones(P, F32))) == apex.ERR_FULL
        check(g, o)
        for nb, k in ((2, 64), (1, 300)):
            rnd = rng.integers(0, U64, nb * k, dtype=np.uint64)
            rco, oo = o.sample(nb, k, 0.5, rnd)
            rcg, go = g.sample(nb, k, 0.5, dev(rnd))
            assert rcg == rco == 0
            torch.cuda.synchronize()
            assert_sample_equal(go, oo)
        keys = np.concatenate([oo["key"], oo["key"][:50], np.array([0, U64 - 1, (5 << 32) | 3], np.uint64)])
        newp = rng.lognormal(0, 1.5, len(keys)).astype(F32)
        newp[:2] = [np.inf, 0.0]
        assert o.update_priorities(keys, newp) == 0
        assert g.update_priorities(dev(keys), dev(newp)) == 0
        check(g, o)
        # more than 1024 pairs: the two-pass update (batches of up to 1024 take one workgroup)
        rnd = rng.integers(0, U64, 4 * 400, dtype=np.uint64)
        rco, oo4 = o.sample(4, 400, 0.5, rnd, payload=False)
        assert rco == 0
        keys4 = np.concatenate([oo4["key"], oo4["key"][:200]])
        newp4 = rng.lognormal(0, 1.5, len(keys4)).astype(F32)
        assert o.update_priorities(keys4, newp4) == 0
        assert g.update_priorities(dev(keys4), dev(newp4)) == 0
        check(g, o)
        e = max(0, o.size - C)
        rnd = rng.integers(0, U64, (rounds, max(e, 1)), dtype=np.uint64)
        rco, eo = o.evict(rounds, rnd)
        rcg, eg = g.evict(rounds, dev(rnd))
        assert (rcg, eg) == (rco, eo) and eo == e
        check(g, o)
        # keys drawn before the eviction: those of evicted transitions are dropped on both sides
        assert o.update_priorities(keys, newp) == 0
        assert g.update_priorities(dev(keys), dev(newp)) == 0
        check(g, o)


def test_rounds_running_out_and_edges():
    from paper_1803_00933_amd import apex
    rng = np.random.default_rng(3)
    g = apex.PeReplay(2, 4, 16, 4, alpha=1.0, alpha_evict=-1.0, eps=0.0)
    o = oracle.PrioritizedEvictionReplay(2, 4, 16, 4, alpha=1.0, alpha_evict=-1.0, eps=0.0)
    prio = np.array([1, 2, 4, 8], F32)
    o.add(prio), g.add(dev(prio))
    # one round, both points inside the heaviest transition: one eviction short (the hand-worked case)
    assert g.evict(1, dev(np.zeros(2, np.uint64))) == (0, 1) == o.evict(1, np.zeros(2, np.uint64))
    check(g, o)
    assert g.evict(3, dev(np.zeros(3, np.uint64))) == (0, 1) == o.evict(3, np.zeros(3, np.uint64))
    check(g, o)
    assert g.evict(3, dev(np.zeros(3, np.uint64))) == (0, 0)
    assert g.sample(1, 4, 0.4, dev(np.zeros(4, np.uint64)))[0] == 0
    empty = apex.PeReplay(2, 4, 16, 4)
    assert empty.sample(1, 4, 0.4, dev(np.zeros(4, np.uint64)))[0] == apex.ERR_EMPTY
    for bad in (dict(alpha_evict=2.0), dict(alpha=float("nan")), dict(eps=-1.0)):
        with pytest.raises(ValueError):
            apex.PeReplay(2, 4, 16, 4, **bad)


def test_control_shape_with_prioritized_eviction():
    """The continuous-control workload as the paper ran it: capacity 1,000,000, sampling exponent 0.6, eviction
    exponent -0.4; add rounds of 64 x 50, batch 512, eviction every 10 rounds."""
    from paper_1803_00933_amd import apex, synth
    w = synth.WORKLOADS["control"]
    g = apex.PeReplay(w.capacity, w.max_slots, w.obs_bytes, w.act_bytes)
    o = oracle.PrioritizedEvictionReplay(w.capacity, w.max_slots, w.obs_bytes, w.act_bytes, payload=False)
    prio = synth.priorities("lognormal1", w.seed, 0, w.capacity, tag="bulk")
    assert o.add(prio)[0] == 0 and g.add(dev(prio)) == 0
    check(g, o)
    rounds = 5
    for step in range(60):
        p_new = synth.priorities("lognormal1", w.seed, step + 1, w.add_count, tag="bulk")
        assert o.add(p_new)[0] == 0 and g.add(dev(p_new)) == 0
        rnd = synth.uniforms(w.seed, step, 1, w.k).reshape(-1)
        rco, oo = o.sample(1, w.k, w.beta, rnd, payload=False)
        rcg, go = g.sample(1, w.k, w.beta, dev(rnd))
        torch.cuda.synchronize()
        assert_sample_equal(go, oo, payload=False)
        newp = synth.priorities(w.td_dist, w.seed, step, w.k)
        assert o.update_priorities(oo["key"], newp) == 0 and g.update_priorities(go["key"], dev(newp)) == 0
        if (step + 1) % 10 == 0:
            e = o.size - w.capacity
            rnd_e = np.random.default_rng(step).integers(0, U64, (rounds, e), dtype=np.uint64)
            assert g.evict(rounds, dev(rnd_e)) == o.evict(rounds, rnd_e) == (0, e)
            check(g, o)
    check(g, o)


def test_control_schedule_without_the_host_in_the_loop():
    """The control-shaped schedule on the memory with prioritized eviction through the calls that wait for nothing:
    an actor round in one launch (n-step priorities + add), a learner step in two (draw; gather + weights +
    write-back), the eviction enqueued - against the oracle doing n-step priorities, add, sample, update, evict."""
    from paper_1803_00933_amd import apex, synth
    w = synth.WORKLOADS["control"]
    g = apex.PeReplay(w.capacity, w.max_slots, w.obs_bytes, w.act_bytes)
    o = oracle.PrioritizedEvictionReplay(w.capacity, w.max_slots, w.obs_bytes, w.act_bytes)
    g.storage.zero_()   # the bulk add names no actions and returns: those columns stay as they are, zero in the oracle
    prio = synth.priorities("lognormal1", w.seed, 0, w.capacity, tag="bulk")
    obs0 = np.zeros((w.capacity, w.obs_bytes), np.uint8)
    assert o.add(prio, obs0)[0] == 0 and g.add(dev(prio), dev(obs0)) == 0
    del obs0
    rounds, steps = 5, 100
    outs = [g.alloc_sample_outputs(1, w.k) for _ in range(steps)]
    refs = []
    key0 = w.capacity
    for step in range(steps):                      # nothing in this loop waits for the GPU (the oracle runs beside it)
        d = synth.actor_round(w, step)
        obs = synth.obs_rows(w.seed, key0, w.add_count, w.obs_bytes)
        ref = oracle.nstep_priorities(d["q_online"], d["q_target"], d["action"], d["reward"], d["discount"],
                                      w.n, w.alpha, w.eps, w.frac_bits, w.max_slots)
        assert o.add(ref[0].reshape(-1), obs, d["act"], ref[1].reshape(-1), ref[2].reshape(-1))[0] == 0
        assert g.add_round(dev(d["q_online"]), dev(d["q_target"]), dev(d["action"]), dev(d["reward"]),
                           dev(d["discount"]), w.n, dev(obs), dev(d["act"])) == 0
        key0 += w.add_count
        rnd = synth.uniforms(w.seed, step, 1, w.k).reshape(-1)
        newp = synth.priorities(w.td_dist, w.seed, step, w.k)
        rco, oo = o.sample(1, w.k, w.beta, rnd)
        assert rco == 0 and o.update_priorities(oo["key"], newp) == 0
        refs.append(oo)
        assert g.sample_update(w.k, w.beta, dev(rnd), dev(newp), outs[step]) == 0
        if (step + 1) % 10 == 0:
            e = o.size - w.capacity
            rnd_e = np.random.default_rng(step).integers(0, U64, (rounds, e), dtype=np.uint64)
            assert o.evict(rounds, rnd_e) == (0, e)
            assert g.evict_enqueue(rounds, dev(rnd_e)) == (0, e)
    torch.cuda.synchronize()
    for step in range(steps):
        assert_sample_equal(outs[step], refs[step])
    check(g, o)
    # the eviction that reports back still agrees, and so does the plain path after the enqueued ones
    p_new = synth.priorities("lognormal1", w.seed, 99, w.add_count, tag="bulk")
    assert o.add(p_new)[0] == 0 and g.add(dev(p_new)) == 0
    e = o.size - w.capacity
    rnd_e = np.random.default_rng(7).integers(0, U64, (rounds, e), dtype=np.uint64)
    assert g.evict(rounds, dev(rnd_e)) == o.evict(rounds, rnd_e) == (0, e)
    check(g, o)


def test_enqueued_eviction_that_falls_short_is_noticed():
    """One round with all points inside one transition removes 1 of the 2 asked for: the host's count is corrected
    from the snapshot the call left behind - an add that only fits if both were gone is refused, the next eviction
    asks for the one that is left - and the device state equals the oracle's throughout."""
    from paper_1803_00933_amd import apex
    g = apex.PeReplay(2, 4, 16, 4, alpha=1.0, alpha_evict=-1.0, eps=0.0)
    o = oracle.PrioritizedEvictionReplay(2, 4, 16, 4, alpha=1.0, alpha_evict=-1.0, eps=0.0)
    prio = np.array([1, 2, 4, 8], F32)
    o.add(prio), g.add(dev(prio))
    assert o.evict(1, np.zeros(2, np.uint64)) == (0, 1)
    assert g.evict_enqueue(1, dev(np.zeros(2, np.uint64))) == (0, 2)     # asked for two
    three = np.array([1, 1, 1], F32)
    assert g.add(dev(three)) == apex.ERR_FULL == o.add(three)[0]         # 3 stored, 4 slots: no room for three
    one = np.array([3], F32)
    assert g.add(dev(one)) == 0 == o.add(one)[0]
    check(g, o)
    assert o.evict(3, np.zeros((3, 2), np.uint64)) == (0, 2)
    assert g.evict_enqueue(3, dev(np.zeros((3, 2), np.uint64))) == (0, 2)
    torch.cuda.synchronize()
    check(g, o)
    assert g.evict_enqueue(3, dev(np.zeros((3, 2), np.uint64))) == (0, 0)
    # limits of the fused calls
    big = apex.PeReplay(10, 16, 8192, 4)
    z = torch.zeros((1, 3, 1), device="cuda:0")
    zi = torch.zeros((1, 3), dtype=torch.int32, device="cuda:0")
    obs = torch.zeros((2, 8192), dtype=torch.uint8, device="cuda:0")
    assert big.add_round(z, z, zi, z[:, :, 0].contiguous(), z[:, :, 0].contiguous(), 1, obs) == apex.ERR_TOO_LARGE
    out = g.alloc_sample_outputs(1, 2000)
    assert g.sample_update(2000, 0.4, dev(np.zeros(2000, np.uint64)), dev(np.zeros(2000, F32)), out) == apex.ERR_TOO_LARGE
    empty = apex.PeReplay(2, 4, 16, 4)
    out = empty.alloc_sample_outputs(1, 4)
    assert empty.sample_update(4, 0.4, dev(np.zeros(4, np.uint64)), dev(np.zeros(4, F32)), out) == apex.ERR_EMPTY


@pytest.mark.parametrize("P,C,ob,ab,S,T,n,A,k", [
    (600, 400, 12, 4, 3, 7, 3, 4, 33),          # rows of three words, one tree level, ragged everything
    (5000, 4000, 7, 3, 5, 11, 2, 1, 100),       # rows of single bytes, critic values
    (70_000, 60_000, 4096, 8, 4, 50, 5, 18, 512),  # the longest rows the fused calls take, three levels
    (9000, 6001, 4096, 4, 61, 41, 3, 4, 64),    # rounds of more workgroups than the chip holds, four transitions each
    (9000, 6001, 1000, 4, 149, 10, 9, 2, 64),   # a last workgroup of 2 of 16 transitions; more steps than are held
])
def test_fused_calls_on_small_and_ragged_shapes(P, C, ob, ab, S, T, n, A, k):
    """apex_pe_add_round / apex_pe_sample_update / apex_pe_evict_enqueue against the oracle's n-step priorities,
    add, sample, update, evict on shapes that take every vector width, with heavy-tailed priorities (repeated
    slots inside a batch) and evictions that need several rounds."""
    from paper_1803_00933_amd import apex, synth
    rng = np.random.default_rng(P + ob)
    g = apex.PeReplay(C, P, ob, ab)
    o = oracle.PrioritizedEvictionReplay(C, P, ob, ab)
    w = synth.WORKLOADS["tiny"].scaled(streams=S, chunk=T, n=n, num_actions=A, act_bytes=ab)
    fill = C - 2 * S * T
    prio = (rng.pareto(0.5, fill) + 1e-3).astype(F32)
    obs = rng.integers(0, 256, (fill, ob), dtype=np.uint8)
    act = rng.integers(0, 256, (fill, ab), dtype=np.uint8)
    ret, gacc = rng.standard_normal(fill).astype(F32), rng.random(fill).astype(F32)
    assert o.add(prio, obs, act, ret, gacc)[0] == 0 and g.add(dev(prio), dev(obs), dev(act), dev(ret), dev(gacc)) == 0
    rounds = 6
    for step in range(12):
        d = synth.actor_round(w, step, with_payload=False)
        d["q_online"] *= F32(3.0)                      # larger TD errors: heavier tails
        obs = rng.integers(0, 256, (S * T, ob), dtype=np.uint8)
        act = rng.integers(0, 256, (S * T, ab), dtype=np.uint8)
        ref = oracle.nstep_priorities(d["q_online"], d["q_target"], d["action"], d["reward"], d["discount"],
                                      n, 0.6, 1e-6, 24, P)
        rco = o.add(ref[0].reshape(-1), obs, act, ref[1].reshape(-1), ref[2].reshape(-1))[0]
        rcg = g.add_round(dev(d["q_online"]), dev(d["q_target"]), dev(d["action"]), dev(d["reward"]),
                          dev(d["discount"]), n, dev(obs), dev(act))
        assert rcg == rco
        rnd = rng.integers(0, U64, k, dtype=np.uint64)
        newp = (rng.pareto(0.5, k) + 1e-3).astype(F32)
        newp[rng.random(k) < 0.1] = 0.0
        rco, oo = o.sample(1, k, 0.7, rnd)
        assert rco == 0 and o.update_priorities(oo["key"], newp) == 0
        out = g.alloc_sample_outputs(1, k)
        assert g.sample_update(k, 0.7, dev(rnd), dev(newp), out) == 0
        torch.cuda.synchronize()
        assert_sample_equal(out, oo)
        if step % 3 == 2:
            e = max(0, o.size - C)
            rnd_e = rng.integers(0, U64, (rounds, max(e, 1)), dtype=np.uint64)
            rco, eo = o.evict(rounds, rnd_e)
            assert g.evict_enqueue(rounds, dev(rnd_e)) == (rco, e)
        check(g, o)


@pytest.mark.parametrize("enqueue", [False, True])
def test_eviction_with_uniforms_for_fewer_than_are_due(enqueue):
    """A program that sizes its uniforms for what it adds meets a larger eviction after one that fell short: the binding
    repeats the words it has, and refuses a tensor that lacks words of the first round; nothing is read past the end."""
    from paper_1803_00933_amd import apex
    rng = np.random.default_rng(3)
    cap, P, n, rounds = 600, 1000, 300, 3
    g = apex.PeReplay(cap, P, 4, 4, alpha_evict=0.4)
    o = oracle.PrioritizedEvictionReplay(cap, P, 4, 4, alpha_evict=0.4)
    prio = rng.lognormal(0, 3.0, cap + n + 7).astype(F32)
    assert o.add(prio)[0] == 0 and g.add(dev(prio)) == 0
    evict = g.evict_enqueue if enqueue else g.evict
    with pytest.raises(ValueError):
        evict(rounds, dev(rng.integers(0, U64, n + 6, dtype=np.uint64)))
    check(g, o)
    rnd = rng.integers(0, U64, (rounds, n), dtype=np.uint64)   # 900 words for 3 x 307
    rco, gone = o.evict(rounds, np.concatenate([rnd.reshape(-1)] * 2))
    rcg, told = evict(rounds, dev(rnd))
    assert (rcg, told) == (rco, n + 7 if enqueue else gone)
    check(g, o)


@pytest.mark.parametrize("e", [1, 1023, 1025, 4097, 65_535, 65_536, 65_537, 70_000])
def test_rounds_at_the_edges_of_the_removal(e):
    """Rounds of whole and ragged workgroups (512 candidates, 1024 above the line), on both sides of the line (65,536) above
    which a launch of its own counts the candidates; heavy-tailed priorities, so that rounds have long runs of equal candidates.
    Two evictions in a row: the second starts from the counters that the first has left."""
    from paper_1803_00933_amd import apex
    rng = np.random.default_rng(e)
    cap, rounds = max(100, e // 2), 3
    P = cap + e
    g = apex.PeReplay(cap, P, 4, 4, alpha_evict=0.4)
    o = oracle.PrioritizedEvictionReplay(cap, P, 4, 4, alpha_evict=0.4)
    for _ in range(2):
        prio = rng.lognormal(0, 3.0, P - o.size).astype(F32)
        assert o.add(prio)[0] == 0
        assert g.add(dev(prio)) == 0
        rnd = rng.integers(0, U64, (rounds, o.size - cap), dtype=np.uint64)
        assert g.evict(rounds, dev(rnd)) == o.evict(rounds, rnd)
        check(g, o)


@pytest.mark.parametrize("k", [1, 63, 64, 65, 128, 129, 1000, 1023, 1024])
@pytest.mark.parametrize("weights", [True, False])
def test_write_back_at_the_edges_of_its_waves(k, weights):
    """apex_pe_sample_update for batches around the waves' shares of 64 pairs, on few transitions of which some are drawn
    again and again, across the shares too (the last pair of a slot stands)."""
    from paper_1803_00933_amd import apex
    rng = np.random.default_rng(k)
    C, P = 700, 900
    g, o = apex.PeReplay(C, P, 20, 4), oracle.PrioritizedEvictionReplay(C, P, 20, 4)
    prio = (rng.pareto(0.5, C) + 1e-3).astype(F32)
    obs, act = (rng.integers(0, 256, (C, n), dtype=np.uint8) for n in (20, 4))
    ret, gacc = rng.standard_normal(C).astype(F32), rng.random(C).astype(F32)
    assert o.add(prio, obs, act, ret, gacc)[0] == 0 and g.add(dev(prio), dev(obs), dev(act), dev(ret), dev(gacc)) == 0
    for it in range(4):
        rnd = rng.integers(0, U64, k, dtype=np.uint64)
        newp = (rng.pareto(0.5, k) + 1e-3).astype(F32)
        newp[rng.random(k) < 0.1] = np.inf
        rco, oo = o.sample(1, k, 0.7, rnd)
        assert rco == 0 and o.update_priorities(oo["key"], newp) == 0
        out = g.alloc_sample_outputs(1, k)
        if not weights:
            out["weight"] = None
        assert g.sample_update(k, 0.7, dev(rnd), dev(newp), out) == 0
        torch.cuda.synchronize()
        if not weights:
            out["weight"] = torch.from_numpy(oo["weight"].astype(F32))
        assert_sample_equal(out, oo)
        check(g, o)


@pytest.mark.parametrize("ob,ab", [(15, 1), (16, 3), (17, 4), (28, 5), (272, 32), (256, 33), (1040, 64), (4096, 67), (12, 1100)])
def test_adds_and_steps_around_the_pieces_of_a_row(ob, ab):
    """apex_pe_add with and without its columns and apex_pe_sample_update, for rows and action bytes around the units they
    are moved in, and numbers of transitions around a wave's and a workgroup's share."""
    from paper_1803_00933_amd import apex
    rng = np.random.default_rng(ob * 3 + ab)
    P = 3100
    g, o = apex.PeReplay(P, P, ob, ab), oracle.PrioritizedEvictionReplay(P, P, ob, ab)
    for n, columns in ((300, True), (1, True), (63, False), (64, True), (65, False), (257, True), (1000, True), (1025, False)):
        prio = rng.lognormal(0, 1, n).astype(F32)
        obs, act = (rng.integers(0, 256, (n, m), dtype=np.uint8) for m in (ob, ab))
        ret, gacc = rng.standard_normal(n).astype(F32), rng.random(n).astype(F32)
        assert o.add(prio, obs, act, ret, gacc)[0] == 0
        if not columns:       # written in place by their producer
            first = o.inserted - n
            at = torch.arange(first, first + n, device="cuda:0")
            lay = g.layout
            for off, size, x in ((lay.act_offset, ab, act), (lay.ret_offset, 4, ret), (lay.gacc_offset, 4, gacc)):
                g.storage[off:off + P * size].view(P, size)[at] = dev(x.view(np.uint8).reshape(n, size))
            act = ret = gacc = None
        assert g.add(*(None if x is None else dev(x) for x in (prio, obs, act, ret, gacc))) == 0
        k = int(rng.integers(1, 200))
        rnd, newp = rng.integers(0, U64, k, dtype=np.uint64), rng.lognormal(0, 1, k).astype(F32)
        rco, oo = o.sample(1, k, 0.4, rnd)
        assert rco == 0 and o.update_priorities(oo["key"], newp) == 0
        out = g.alloc_sample_outputs(1, k)
        assert g.sample_update(k, 0.4, dev(rnd), dev(newp), out) == 0
        torch.cuda.synchronize()
        assert_sample_equal(out, oo)
        check(g, o)


@pytest.mark.parametrize("e", [63, 64, 65, 511, 512, 513, 2559, 2561, 8191, 8192, 8193, 8704, 8705, 16_384, 16_385, 16_897])
def test_removals_around_a_workgroup_that_counts_for_itself(e):
    """Workgroups of 512 candidates, each counting what lies before it four words at a time and four loads ahead: rounds that
    end a wave and a workgroup, and whose last workgroup has just under, exactly and just over one and two turns of those loads
    (8192 candidates each) before it, with half of the candidates equal to their neighbours."""
    test_rounds_at_the_edges_of_the_removal(e)


@pytest.mark.parametrize("m", [1, 63, 65, 512, 1000, 1024])
def test_updates_of_one_workgroup(m):
    """apex_pe_update_priorities of up to 1024 pairs: slots named again and again (the last pair stands), keys of earlier
    generations and keys of no slot."""
    from paper_1803_00933_amd import apex
    rng = np.random.default_rng(m)
    C, P = 500, 900
    g, o = apex.PeReplay(C, P, 4, 4), oracle.PrioritizedEvictionReplay(C, P, 4, 4)
    stale = np.empty(0, np.uint64)
    for it in range(3):
        prio = rng.lognormal(0, 2.0, P - o.size).astype(F32)
        assert o.add(prio)[0] == 0 and g.add(dev(prio)) == 0
        drawn = o.sample(1, m, 0.4, rng.integers(0, U64, m, dtype=np.uint64))[1]["key"]
        keys = np.where(rng.random(m) < 0.1, np.uint64(P + 3), drawn)
        if len(stale):
            keys = np.where(rng.random(m) < 0.2, rng.choice(stale, m), keys)
        newp = (rng.pareto(0.5, m) + 1e-3).astype(F32)
        newp[rng.random(m) < 0.1] = np.inf
        assert o.update_priorities(keys, newp) == 0 and g.update_priorities(dev(keys), dev(newp)) == 0
        check(g, o)
        stale = drawn
        rnd = rng.integers(0, U64, (3, o.size - C), dtype=np.uint64)
        assert g.evict(3, dev(rnd)) == o.evict(3, rnd)
        check(g, o)
