"""The work that users of the replay memory have it do, as measurable cases.

A case is a dict of plain values.  Five kinds of program are covered, each through the entry points of
``paper_1803_00933_amd.apex`` that such a program calls:

``learner``   a learner on the plain verbs: sample one or several batches (draw, importance weights, gather), then
              write the new priorities back, given (``update``) or recomputed from its Q-values (``from_q``)
``actors``    the actors' side on the plain verbs: n-step priorities of a round, add, evict what is above capacity
``round``     both on one stream: an actor round, then learner steps, then the eviction
``pipeline``  the prefetch pipeline: add rounds beside learner steps, eviction at the end of the period; with
              ``raw_bytes`` the observations go through the block codec
``pe``        the memory with prioritized eviction: rounds of (add round, learner step), then an eviction

Sizes are those of the workloads in ``synth.WORKLOADS`` and of the paper's own feature observations (67 floats,
actions of 21), or generic odd ones.  ``draw`` spreads the same kinds over the ranges in between.
"""
import math

import torch

from paper_1803_00933_amd import apex

DEVICE = "cuda:0"
ALPHA, ALPHA_EVICT, BETA, EPS, FRAC_BITS, GAMMA = 0.6, -0.4, 0.4, 1e-6, 24, 0.99
# a learner's successive calls come with successive uniforms: this many sets of them, so that the rows of one pass
# are not those of the pass before (and do not sit in a cache because of it)
POOL = 64
RING_LIMIT = 8 << 30  # bytes of observations in a drawn case's ring


def _case(name, kind, capacity, slots, obs_bytes, act_bytes, **more):
    c = dict(kind=kind, capacity=capacity, slots=slots, obs_bytes=obs_bytes, act_bytes=act_bytes, k=0, batches=1,
             steps=0, rounds=0, streams=0, chunk=0, n=3, actions=18, priorities="lognormal1", write="update", sets=6,
             raw_bytes=0, flat_share=0.0, evict_rounds=0)
    c.update(more)
    if name:
        c["name"] = name
    return c


def listed():
    frames = 84 * 84 * 4
    return [
        # the smallest memory: one batch of 32 short rows, latency and launches only
        _case("small_step", "learner", 4096, 8192, 32, 4, k=32, actions=4, priorities="absnormal"),
        # continuous control as the paper sizes it: 67-float observations, 21-float actions, batches of 256, critic
        # values as the learner's Q-values
        _case("features_step", "learner", 1_000_000, 1 << 20, 67 * 4, 21 * 4, k=256, actions=1, n=5, write="from_q"),
        # opaque records of an odd length, an odd batch, a ring that is no power of two
        _case("odd_records_step", "learner", 100_003, 110_017, 5003, 7, k=333, batches=3),
        # frame stacks, 2,000,000 of them: one batch of 512, new priorities from the learner's Q-values
        _case("frames_step", "learner", 2_000_000, 1 << 21, frames, 4, k=512, write="from_q"),
        # the learner's prefetch depth as the unit of work: 16 batches of 512 frame stacks per call
        _case("frames_prefetch", "pipeline", 250_000, 1 << 18, frames, 4, k=512, batches=16, steps=4, sets=2),
        # an actor round of 360 x 50 frame stacks: n-step priorities, payload and masses, eviction
        _case("frames_actors", "actors", 100_000, 1 << 17, frames, 4, streams=360, chunk=50),
        # one period of the paper's Atari schedule: 100 learner steps, an add round every 25, eviction at the end
        _case("frames_period", "pipeline", 2_000_000, 1 << 21, frames, 4, k=512, steps=25, rounds=4, streams=360,
              chunk=50),
        # half a period with observations stored through the codec, game-like screens (most blocks flat)
        _case("codec_period", "pipeline", 200_000, 1 << 18, 0, 4, k=512, steps=25, rounds=2, streams=360,
              chunk=50, raw_bytes=frames, flat_share=0.8),
        # continuous control through the pipeline: a small add round before every learner step
        _case("control_period", "pipeline", 1_000_000, 1 << 20, 256, 32, k=512, steps=1, rounds=10, streams=64,
              chunk=50, n=5, actions=1),
        # heavy-tailed priorities, 16 batches of 512 short rows per call, all 8192 priorities written back
        _case("skewed_prefetch", "pipeline", 1 << 21, 1 << 21, 64, 4, k=512, batches=16, steps=4, sets=4,
              priorities="pareto"),
        # the largest memory: 2^24 transitions, an actor round of 1024 x 50, a batch of 4096
        _case("large_memory_round", "round", 1 << 24, (1 << 24) + (1 << 20), 128, 4, k=4096, steps=4, streams=1024,
              chunk=50, priorities="lognormal2"),
        # the memory with prioritized eviction as the paper runs it: ten rounds of 64 x 50, ten learner steps, then the
        # excess of 32,000 evicted by priority
        _case("priority_eviction_period", "pe", 1_000_000, (1 << 20) + (1 << 16), 256, 32, k=512, rounds=10, streams=64,
              chunk=50, n=5, actions=1, evict_rounds=3),
    ]


# ---------------------------------------------------------------------------------------------------------------------
# drawn cases
# ---------------------------------------------------------------------------------------------------------------------

def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _row_bytes(rng, lo, hi):
    """Mostly whole floats or whole 16-byte pieces, sometimes any number of bytes."""
    v = _log_int(rng, lo, hi)
    step = rng.choice([16, 16, 4, 4, 1])
    return max(step, v // step * step)


def draw(rng):
    kind = rng.choice(["learner", "learner", "actors", "round", "pipeline", "pipeline", "pe"])
    dist = rng.choice(["absnormal", "lognormal1", "lognormal2", "pareto"])
    actions, n = rng.choice([1, 2, 4, 6, 18]), rng.choice([1, 3, 5])
    act_bytes = rng.choice([1, 4, 4, 8, 32, 84])
    common = dict(priorities=dist, actions=actions, n=n)
    if kind == "learner":
        obs = _row_bytes(rng, 16, 32768)
        cap = _log_int(rng, 3000, min(1 << 24, RING_LIMIT // obs))
        k = _log_int(rng, 16, 4096)
        batches = rng.choice([1, 1, 1, 2, 5, 16]) if k <= 600 else 1
        return _case(None, kind, cap, cap + rng.randrange(0, cap // 8), obs, act_bytes, k=k, batches=batches,
                     write=rng.choice(["update", "from_q"]), **common)
    streams, chunk = _log_int(rng, 8, 1024), rng.randrange(20, 61)
    count = streams * chunk
    if kind in ("actors", "round"):
        obs = _row_bytes(rng, 16, min(28224, (2 << 30) // (4 * count)))
        cap = _log_int(rng, 2 * count, max(3 * count, min(1 << 24, (3 << 30) // obs)))
        more = {}
        if kind == "round":
            more = dict(k=_log_int(rng, 16, 4096), steps=rng.randrange(1, 5), write=rng.choice(["update", "from_q"]))
        return _case(None, kind, cap, cap + count + rng.randrange(0, count), obs, act_bytes, streams=streams,
                     chunk=chunk, **more, **common)
    if kind == "pipeline":
        form = rng.choice(["batch", "batch", "prefetch", "codec"])
        if form == "prefetch":
            obs = _row_bytes(rng, 32, 28224)
            cap = _log_int(rng, 20000, min(1 << 22, RING_LIMIT // obs))
            return _case(None, kind, cap, cap + rng.randrange(0, cap // 8), obs, act_bytes, k=_log_int(rng, 128, 600),
                         batches=rng.randrange(4, 17), steps=rng.randrange(1, 5), sets=rng.choice([2, 4]), **common)
        raw = 64 * _log_int(rng, 8, 441) if form == "codec" else 0
        obs = 0 if raw else _row_bytes(rng, 16, 28224)
        size = raw * 9 // 8 + 64 if raw else obs
        rounds = rng.randrange(1, 5)
        streams = max(8, min(streams, 400))
        count = streams * chunk
        cap = _log_int(rng, max(20000, 4 * count), max(30000, 6 * count, min(1 << 21, RING_LIMIT // size)))
        return _case(None, kind, cap, cap + rounds * count + rng.randrange(0, count), obs, act_bytes,
                     k=_log_int(rng, 32, 1024), steps=rng.randrange(1, 26), rounds=rounds, streams=streams, chunk=chunk,
                     raw_bytes=raw, flat_share=round(rng.uniform(0.0, 0.95), 2) if raw else 0.0, **common)
    streams = max(8, min(streams, 128))
    count, rounds = streams * chunk, rng.randrange(2, 11)
    obs = 4 * _log_int(rng, 4, 250)
    cap = _log_int(rng, max(20000, 2 * rounds * count), 1 << 20)
    return _case(None, kind, cap, cap + rounds * count + rng.randrange(0, count), obs, act_bytes,
                 k=_log_int(rng, 32, 1024), rounds=rounds, streams=streams, chunk=chunk, evict_rounds=3, **common)


# ---------------------------------------------------------------------------------------------------------------------
# what a program has in hand before the call
# ---------------------------------------------------------------------------------------------------------------------

def _priorities(dist, shape, gen):
    """|TD error|-like values of the distributions that synth.priorities names."""
    if dist == "pareto":  # Pareto(1.1), a fifth of them zero
        u = torch.rand(shape, device=DEVICE, generator=gen).clamp_(min=1e-7)
        p = u.pow_(-1.0 / 1.1)
        return torch.where(torch.rand(shape, device=DEVICE, generator=gen) < 0.2, torch.zeros_like(p), p)
    z = torch.randn(shape, device=DEVICE, generator=gen)
    return z.abs_() if dist == "absnormal" else z.mul_(2.0 if dist == "lognormal2" else 1.0).exp_()


def _uniforms(shape, gen):
    """64-bit uniforms: two 32-bit halves (torch's integers end at 2^63)."""
    hi, lo = (torch.randint(0, 1 << 32, shape, dtype=torch.int64, device=DEVICE, generator=gen) for _ in range(2))
    return (hi << 32) | lo


def _random_bytes(view, gen):
    """Fills a contiguous uint8 view."""
    flat = view.reshape(-1)
    whole = flat.numel() // 8 * 8
    piece = 1 << 31
    for at in range(0, whole, piece):
        flat[at:min(at + piece, whole)].view(torch.int64).random_(-(1 << 63), None, generator=gen)
    if whole < flat.numel():
        flat[whole:].random_(0, 256, generator=gen)


def _screens(count, raw_bytes, flat_share, gen):
    """Rows like game screens: a 64-byte block is one of 8 background bytes with probability flat_share."""
    rows = torch.empty((count, raw_bytes // 64, 64), dtype=torch.uint8, device=DEVICE)
    _random_bytes(rows, gen)
    flat = torch.rand((count, raw_bytes // 64, 1), device=DEVICE, generator=gen) < flat_share
    pal = (torch.randint(0, 8, (count, raw_bytes // 64, 1), device=DEVICE, generator=gen) * 31).to(torch.uint8)
    return torch.where(flat, pal, rows).view(count, raw_bytes)


def _actor_inputs(case, obs_bytes, gen):
    S, L, A = case["streams"], case["chunk"] + case["n"], case["actions"]
    count = S * case["chunk"]
    d = dict(q_online=torch.randn((S, L, A), device=DEVICE, generator=gen),
             q_target=torch.randn((S, L, A), device=DEVICE, generator=gen),
             action=torch.randint(0, A, (S, L), device=DEVICE, generator=gen).to(torch.int32),
             reward=torch.randn((S, L), device=DEVICE, generator=gen))
    done = torch.rand((S, L), device=DEVICE, generator=gen) < 0.05
    d["discount"] = torch.where(done, 0.0, GAMMA).to(torch.float32)
    d["act"] = torch.empty((count, case["act_bytes"]), dtype=torch.uint8, device=DEVICE)
    _random_bytes(d["act"], gen)
    if case["raw_bytes"]:
        d["obs"] = _screens(count, case["raw_bytes"], case["flat_share"], gen)
    else:
        d["obs"] = torch.empty((count, obs_bytes), dtype=torch.uint8, device=DEVICE)
        _random_bytes(d["obs"], gen)
    for name in ("prio", "ret", "gacc"):
        d[name] = torch.empty((S, case["chunk"]), dtype=torch.float32, device=DEVICE)
    return d


def _fill(case, rep, gen):
    """Brings the memory to its capacity."""
    left, dist = case["capacity"], case["priorities"]
    if case["kind"] != "pe":
        _random_bytes(rep.act_view(), gen)
        rep.ret_view().normal_(generator=gen)
        rep.gacc_view().fill_(GAMMA ** case["n"])
    if case["raw_bytes"]:  # through the encoder
        rows = _screens(min(left, 16384), case["raw_bytes"], case["flat_share"], gen)
        while left:
            n = min(left, rows.shape[0])
            assert rep.add_payload_encoded(rows[:n]) == apex.OK
            assert rep.add_publish(_priorities(dist, (n,), gen))[0] == apex.OK
            left -= n
        return
    _random_bytes(rep.obs_view(), gen)  # rows written in place, then published
    while left:
        n = min(left, 1 << 22)
        prio = _priorities(dist, (n,), gen)
        if case["kind"] == "pe":
            act = torch.empty((n, case["act_bytes"]), dtype=torch.uint8, device=DEVICE)
            _random_bytes(act, gen)
            ret = torch.randn(n, device=DEVICE, generator=gen)
            assert rep.add(prio, None, act, ret, torch.full_like(ret, GAMMA ** case["n"])) == apex.OK
        else:
            assert rep.add(prio)[0] == apex.OK
        left -= n


def prepare(case, seed):
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)
    kind, k, nb, A = case["kind"], case["k"], case["batches"], case["actions"]
    obs_bytes = int(apex.lib.apex_codec_row_bytes(case["raw_bytes"])) if case["raw_bytes"] else case["obs_bytes"]
    state = dict(case=case, turn=0)
    if case["streams"]:
        state["actors"] = _actor_inputs(case, obs_bytes, gen)
    if kind == "pe":
        rep = apex.PeReplay(case["capacity"], case["slots"], obs_bytes, case["act_bytes"], ALPHA, ALPHA_EVICT, EPS,
                            FRAC_BITS)
        count = case["streams"] * case["chunk"]
        state["evict_rnd"] = _uniforms((case["evict_rounds"], case["rounds"] * count), gen)
        state["out"] = [rep.alloc_sample_outputs(1, k) for _ in range(2)]
        state["rnd"] = _uniforms((POOL, k), gen)
        state["prio"] = _priorities(case["priorities"], (POOL, k), gen)
    else:
        rep = apex.Replay(case["capacity"], case["slots"], obs_bytes, case["act_bytes"], ALPHA, EPS, FRAC_BITS)
        if kind == "pipeline":
            state["pipe"] = apex.Pipeline(rep, case["sets"], nb, k)
            if case["raw_bytes"]:
                assert state["pipe"].set_codec(case["raw_bytes"]) == apex.OK
            # every steps call of a pass has uniforms of its own, and the pass after that others again
            calls = max(1, case["rounds"])
            turns = max(1, min(8, 256 // (calls * case["steps"])))
            state["rnd"] = _uniforms((turns, calls, case["steps"], nb * k), gen)
            state["prio"] = _priorities(case["priorities"], (turns, calls, case["steps"], nb * k), gen)
        elif kind != "actors":
            state["out"] = rep.alloc_sample_outputs(nb, k)
            state["rnd"] = _uniforms((POOL, nb * k), gen)
            if case["write"] == "update":
                state["prio"] = _priorities(case["priorities"], (POOL, nb * k), gen)
            else:
                state["q"] = [(torch.randn(nb * k, device=DEVICE, generator=gen),
                               torch.randn((nb * k, A), device=DEVICE, generator=gen),
                               torch.randn((nb * k, A), device=DEVICE, generator=gen)) for _ in range(4)]
                state["prio_out"] = torch.empty(nb * k, device=DEVICE)
    state["rep"] = rep
    _fill(case, rep, gen)
    return state


# ---------------------------------------------------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------------------------------------------------

def _learner_step(state, case):
    rep, out, i = state["rep"], state["out"], state["turn"]
    state["turn"] = i + 1
    rc, _ = rep.sample(case["batches"], case["k"], BETA, state["rnd"][i % POOL], out=out)
    assert rc == apex.OK, rc
    if case["write"] == "update":
        rc = rep.update_priorities(out["key"], state["prio"][i % POOL])
    else:
        taken, online, target = state["q"][i % 4]
        rc = rep.update_from_q(out["key"], taken, online, target, state["prio_out"])
    assert rc == apex.OK, rc


def _actor_round(state, case):
    rep, a = state["rep"], state["actors"]
    rc, prio, ret, gacc, _ = apex.nstep_priorities(
        a["q_online"], a["q_target"], a["action"], a["reward"], a["discount"], case["n"], ALPHA, EPS, FRAC_BITS,
        case["slots"], want_fx=False, out=(a["prio"], a["ret"], a["gacc"], None))
    assert rc == apex.OK, rc
    rc, _ = rep.add(prio.view(-1), a["obs"], a["act"], ret.view(-1), gacc.view(-1))
    assert rc == apex.OK, rc


def _rows(view, first, count):
    """Ring rows of the keys [first, first + count)."""
    at, size = first % view.shape[0], view.shape[0]
    return [view[at:min(at + count, size)], view[:max(0, at + count - size)]]


def _batches(outs):
    return [{n: o[n] for n in ("key", "slot", "weight", "obs", "act", "ret", "gacc")} for o in outs]


def _memory(rep):
    """What the memory holds apart from the observations."""
    return dict(mass=rep.level_view(0), act=rep.act_view(), ret=rep.ret_view(), gacc=rep.gacc_view())


def _run_pipeline(state, case):
    rep, pipe = state["rep"], state["pipe"]
    turn = state["turn"] % state["rnd"].shape[0]
    state["turn"] += 1
    rnd, prio = state["rnd"][turn], state["prio"][turn]
    assert pipe.fork() == apex.OK
    if not case["rounds"]:
        rc, _ = pipe.steps(case["steps"], BETA, rnd[0], prio[0])
        assert rc == apex.OK, rc
    for r in range(case["rounds"]):
        a = state["actors"]
        rc = pipe.add_begin(a["q_online"], a["q_target"], a["action"], a["reward"], a["discount"], case["n"], a["obs"],
                            a["act"], a["prio"], a["ret"], a["gacc"])
        assert rc == apex.OK, rc
        rc, _ = pipe.steps(case["steps"], BETA, rnd[r], prio[r])
        assert rc == apex.OK, rc
        rc, first, _ = pipe.add_end(evict=r + 1 == case["rounds"])
        assert rc == apex.OK, rc
    assert pipe.join() == apex.OK
    res = dict(batches=_batches(pipe.sets), mass=rep.level_view(0))
    if case["rounds"] and not case["raw_bytes"]:  # (an encoded row holds bytes that nothing defines)
        res["added"] = _rows(rep.obs_view(), first, case["streams"] * case["chunk"])
    return res


def _run_pe(state, case):
    rep, a = state["rep"], state["actors"]
    for _ in range(case["rounds"]):
        i = state["turn"]
        state["turn"] = i + 1
        rc = rep.add_round(a["q_online"], a["q_target"], a["action"], a["reward"], a["discount"], case["n"], a["obs"],
                           a["act"])
        assert rc == apex.OK, rc
        rc = rep.sample_update(case["k"], BETA, state["rnd"][i % POOL], state["prio"][i % POOL], state["out"][i % 2])
        assert rc == apex.OK, rc
    rc, _ = rep.evict_enqueue(case["evict_rounds"], state["evict_rnd"])
    assert rc == apex.OK, rc
    return dict(batches=_batches(state["out"]), mass=rep.level_view(0), evict_mass=rep.level_view(0, evict_tree=True),
                generation=rep.gen_view(), free=rep.free_ring_view(), obs=rep.obs_view())


def run(state):
    case = state["case"]
    kind, rep = case["kind"], state["rep"]
    if kind == "pipeline":
        return _run_pipeline(state, case)
    if kind == "pe":
        return _run_pe(state, case)
    if kind in ("actors", "round"):
        _actor_round(state, case)
    for _ in range(1 if kind == "learner" else case["steps"]):
        _learner_step(state, case)
    if kind in ("actors", "round"):
        rc, _ = rep.evict()
        assert rc == apex.OK, rc
    res = dict(mass=rep.level_view(0))
    if kind != "actors":
        res["batch"] = _batches([state["out"]])
        if "prio_out" in state:
            res["prio"] = state["prio_out"]
    if kind != "learner":
        res.update(_memory(rep), obs=rep.obs_view())
    return res


# ---------------------------------------------------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------------------------------------------------

def work(case):
    """Bytes: payload read and written once, small outputs and inputs once, and in the sum tree one node per
    (binary) level read for a draw, one read and written for a change of mass."""
    depth = math.ceil(math.log2(case["slots"]))
    small = case["act_bytes"] + 8  # action bytes, partial return, accumulated discount
    row = obs = case["obs_bytes"]
    kept = obs  # bytes of a stored observation that carry data
    if case["raw_bytes"]:
        row = case["raw_bytes"]
        blocks = row // 64
        kept = blocks / 8 + blocks * (case["flat_share"] + 64 * (1 - case["flat_share"]))
    draw_bytes = row + kept + 2 * small + 8 + 16 + 8 * depth  # + uniform; key, slot, weight
    write_bytes = 12 + 16 * (depth + 1)
    if case["write"] == "from_q":
        write_bytes += 4 * (1 + case["actions"]) + 4 + 8
    trees = 2 if case["kind"] == "pe" else 1  # sampling and eviction masses
    add_bytes = row + kept + 2 * small + trees * 16 * (depth + 1) + 4 * (2 * case["actions"] + 3)
    evict_bytes = trees * 16 * (depth + 1) + (8 * depth + 12 if trees == 2 else 0)
    kind, count, samples = case["kind"], case["streams"] * case["chunk"], case["k"] * case["batches"]
    if kind == "learner":
        steps, adds = 1, 0
    elif kind == "actors":
        steps, adds = 0, count
    elif kind == "round":
        steps, adds = case["steps"], count
    elif kind == "pe":
        steps, adds = case["rounds"], case["rounds"] * count
    else:
        steps, adds = case["steps"] * max(1, case["rounds"]), case["rounds"] * count
    total = steps * samples * (draw_bytes + trees * write_bytes) + adds * (add_bytes + evict_bytes)
    return {"bytes": float(total), "flops": 0.0}


def tolerance(case):
    """Masses, keys, slots and payload are whole numbers and bytes: the same.  Floating outputs are n-step returns and
    importance weights in fp32; the weights' power is within 6e-8 of fp64 in 2-norm and 2.3e-7 of the value at worst
    (ratios of masses over ten decades, exponent 0.4)."""
    return {"rel": 2.5e-7, "max": 1e-6, "differ": 0.0}
