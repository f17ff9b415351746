"""Which launches the library makes and how they are ordered, on a HIP runtime that only records them (no GPU)."""
import recorded_hip


# 6.8 MB of observations: a round whose payload the copy stream carries.
FORKS = """
r = replay(4000, 28224, filled=2000)
p, (tree, add) = pipeline(r, 3, 1, 64)
A, B = 0x1000, 0x2000
hip_calls, had = [], {}

def work(stream, name):      # the caller's stream has new work behind which nothing of its own is ordered
    hip_calls.extend(take())
    hip_calls.append(["mark", stream, name])

%s
assert add_begin(p, 1, 240) == 0 and steps(p, 2) == 0 and add_end(p) == 0
hip_calls.extend(take())
after, out = seen(hip_calls, had)
result = [dict(stream="tree" if c[1] == tree else "add", kernel=c[5], behind=sorted(b)) for c, b in out]
"""


def check_forks(tmp_path, forks, names):
    out = recorded_hip.run(tmp_path, FORKS % forks)
    assert {x["stream"] for x in out} == {"tree", "add"}
    for x in out:
        assert set(names) <= set(x["behind"]), x


def test_a_fork_is_waited_for_by_every_stream_that_is_used(tmp_path):
    check_forks(tmp_path, 'work(A, "a")\nassert call("apex_pipeline_fork", p, A) == 0', ["a"])


def test_forks_behind_two_streams(tmp_path):
    check_forks(tmp_path, 'for s, n in ((A, "a"), (B, "b")):\n'
                          '    work(s, n)\n    assert call("apex_pipeline_fork", p, s) == 0', ["a", "b"])


def test_forks_behind_two_streams_of_one_handle(tmp_path):
    """A stream that is destroyed, and one created later that gets the same handle, are two streams."""
    check_forks(tmp_path, 'for n in ("a", "b"):\n'
                          '    work(A, n)\n    assert call("apex_pipeline_fork", p, A) == 0', ["a", "b"])


def test_many_forks_before_a_copy_stream_is_used(tmp_path):
    check_forks(tmp_path, 'for i in range(20):\n'
                          '    work(A + 16 * (i % 3), str(i))\n'
                          '    assert call("apex_pipeline_fork", p, A + 16 * (i % 3)) == 0', [str(i) for i in range(20)])


def test_forks_of_a_pipeline_that_uses_no_copy_stream_cost_no_waits(tmp_path):
    """Small steps, fork and join again and again: the copy stream, which has nothing to do, is asked to wait for nothing
    once the forks are complete, and for each fork at most once where they are not."""
    for complete in (1, 0):
        out = recorded_hip.run(tmp_path, """
r = replay(4000, 64)
p, (tree, add) = pipeline(r, 3, 1, 64)
C.c_int.in_dll(hip, "complete").value = %d
for i in range(50):
    assert call("apex_pipeline_fork", p, 0x1000) == 0 and steps(p, 1) == 0 and call("apex_pipeline_join", p, 0x1000) == 0
result = [c for c in take() if c[0] == "wait" and c[1] == add]
""" % complete)
        assert len(out) <= (0 if complete else 50)


def test_forks_ask_for_events_in_a_way_that_no_capture_forbids(tmp_path):
    """While any thread of the program captures in the global mode, asking whether an event is complete is refused to every
    other thread, and to the capturing one at the price of its capture, unless the asking thread is in the relaxed mode (2)."""
    queries, mode = recorded_hip.run(tmp_path, """
r = replay(4000, 64)
p, (tree, add) = pipeline(r, 3, 1, 64)
for i in range(50):
    C.c_int.in_dll(hip, "complete").value = i & 1
    assert call("apex_pipeline_fork", p, 0x1000) == 0
result = [[c for c in take() if c[0] == "query"], C.c_int.in_dll(hip, "capture_mode").value]
""")
    assert all(c[2] == 2 for c in queries) and mode == 0, (queries, mode)


def test_a_fork_in_the_callers_own_capture_takes_the_copy_streams_along(tmp_path):
    """All streams of the pipeline enter a capture of the caller's and are joined back, and what is waited for after it
    has nothing of it."""
    out = recorded_hip.run(tmp_path, """
r = replay(4000, 28224, filled=2000)
p, (tree, add) = pipeline(r, 3, 1, 64)
capturing = C.c_int.in_dll(hip, "capturing")
capturing.value = 1
assert call("apex_pipeline_fork", p, 0x1000) == 0 and steps(p, 1) == 0 and call("apex_pipeline_join", p, 0x1000) == 0
capturing.value = 0
captured = take()
assert call("apex_pipeline_fork", p, 0x1000) == 0 and add_begin(p, 1, 240) == 0
result = [captured, take(), tree, add]
""")
    captured, later, tree, add = out
    records, waits = {}, []
    for c in captured:
        if c[0] == "record":
            records[c[1]] = c[2]
        elif c[0] == "wait":
            waits.append((c[1], records[c[2]]))
    assert sorted(waits) == sorted([(tree, 0x1000), (add, 0x1000), (0x1000, tree), (0x1000, add)])
    assert [c[2] for c in later if c[0] == "wait" and c[1] == add][:1] == [c[1] for c in later if c[0] == "record"][:1]
    assert not set(records) & {c[2] for c in later if c[0] == "wait"}


MULTI = """
out = []
for slots, nb, k, depth, n in %r:
    r = replay(slots, 64, filled=slots if slots < 1 << 20 else 1 << 20)
    p, streams = pipeline(r, depth, nb, k)
    assert steps(p, n) == 0
    out.append(launches())
    assert call("apex_pipeline_destroy", p) == 0 and call("apex_replay_destroy", r) == 0
result = out
"""


def multi_launches(tmp_path, shapes):
    """Per shape (slots, batches, samples per batch, sets, steps of the call): the launches of multi_step_kernel, none where
    the steps go another way."""
    return [[x for x in launches if "multi_step" in x["kernel"]] for launches in recorded_hip.run(tmp_path, MULTI % (shapes,))]


def test_weights_of_large_batches_are_shared_out(tmp_path):
    """A step's launch has workgroups for 16 draws, 16 rows and 512 weights each, whatever the size of its batches."""
    shapes = [(1 << 21, nb, k, 2, 3) for nb, k in ((1, 1025), (1, 4096), (1, 16_384), (1, 32_768), (2, 513), (3, 512), (2, 8192))]
    for (_, nb, k, _, n), found in zip(shapes, multi_launches(tmp_path, shapes)):
        parts = nb * -(-k // 16), -(-nb * k // 16), nb * -(-k // 512)
        assert [x["grid"] for x in found] == [parts[0]] + [sum(parts)] * (n - 1) + [parts[1] + parts[2]], (nb, k)
        assert all(x["block"] == 256 for x in found)


def test_steps_of_many_batches_are_two_launches_each(tmp_path):
    """What a drawn sample is held against grows with the number of batches: beyond a number of them two launches do less."""
    shapes = [(1 << 21, nb, k, 2, 2) for nb, k in ((128, 64), (160, 32), (161, 32), (256, 64), (512, 16), (1024, 1), (1024, 32))]
    assert [bool(x) for x in multi_launches(tmp_path, shapes)] == [True, True] + [False] * 5


def test_steps_that_would_crowd_the_top_level_are_two_launches_each(tmp_path):
    """Levels of 300,000 slots: 4688 and 74 nodes; of 2^19: 8192 and 128; of 2^21: 32,768 and 512."""
    shapes = [(slots, nb, k, 2, 2) for slots, nb, k in (
        (300_000, 8, 512), (300_000, 16, 512), (300_000, 1, 4736), (300_000, 1, 4737), (1 << 19, 16, 512), (1 << 19, 17, 512),
        (1 << 21, 32, 512), (1 << 21, 1, 32_768), (30, 3, 640), (30, 3, 641))]
    assert [bool(x) for x in multi_launches(tmp_path, shapes)] == [True, False, True, False, True, False, True, True, True, False]


SAMPLES = """
out = []
for obs_bytes, nb, k in %r:
    r = replay(4096, obs_bytes)
    assert call("apex_replay_sample", r, nb, k, 0.4, memory(), memory(), memory(), memory(), memory(), memory(), memory(), memory(),
                None) == 0
    out.append(launches())
    assert call("apex_replay_destroy", r) == 0
result = out
"""


def test_long_rows_are_copied_by_as_many_workgroups_as_they_need(tmp_path):
    """replay.Sample takes a workgroup per sample for rows of up to 96 KB, of more than 512 samples up to 52 KB; beyond, a
    launch of its own copies the rows with a workgroup per 32 KB."""
    shapes = [(ob, nb, k) for ob in (4100, 28_224, 53_000, 65_536, 98_304, 98_305, 112_896, 400_000, 4_000_000)
              for nb, k in ((1, 1), (1, 32), (1, 512), (1, 513), (3, 300))]
    for (ob, nb, k), found in zip(shapes, recorded_hip.run(tmp_path, SAMPLES % (shapes,))):
        by_rows = [x for x in found if "sample_rows_kernel" in x["kernel"]]
        limit = 96 << 10 if nb * k <= 512 else 52 << 10
        assert bool(by_rows) == (ob <= limit), (ob, nb, k)
        if ob > limit:
            assert [x["grid"] for x in found if "copy_rows" in x["kernel"]] == [nb * k * -(-ob // (32 << 10))]


def test_samples_by_rows_fill_the_chip_once(tmp_path):
    """Two pieces per lane only where all workgroups find room at once (32 waves on each of 256 compute units, a workgroup's
    waves on one of them), and rows of one pass in several rounds only for small batches."""
    shapes = [(ob, nb, k) for ob in (5003, 8192, 16_384, 20_000, 24_000, 28_224, 28_688, 30_720, 32_768)
              for nb, k in ((1, 256), (1, 512), (1, 640), (1, 768), (1, 896), (1, 1024), (2, 600), (3, 512), (12, 100))]
    at_once = lambda waves: 256 * (32 // waves)
    for (ob, nb, k), found in zip(shapes, recorded_hip.run(tmp_path, SAMPLES % (shapes,))):
        pieces = -(-ob // 16)
        waves = {n: min(16, 1 + -(-pieces // (64 * n))) for n in (2, 4)}
        by_rows = [x for x in found if "sample_rows_kernel" in x["kernel"]]
        assert bool(by_rows) == (nb * k <= at_once(waves[4]) or k <= 384), (ob, nb, k)
        for x in by_rows:
            n = 2 if nb * k <= at_once(waves[2]) else 4
            assert "sample_rows_kernelILi%d" % n in x["kernel"] and x["block"] == 64 * waves[n], (ob, nb, k)


def test_large_batches_of_rows_below_the_streaming_size_take_16_lanes_a_sample(tmp_path):
    """One batch of more than 768 samples of rows below 1 KB, of more than 832 below 2 KB: draws by 16 lanes; a workgroup per
    sample otherwise."""
    shapes = [(ob, 1, k) for ob in (16, 1023, 1024, 2047, 2048, 4096) for k in (768, 769, 832, 833, 1024)]
    for (ob, nb, k), found in zip(shapes, recorded_hip.run(tmp_path, SAMPLES % (shapes,))):
        limit = 768 if ob < 1024 else 832 if ob < 2048 else 1024
        assert ("sample_rows_kernel" in found[0]["kernel"]) == (k <= limit), (ob, k)


def test_large_batches_are_gathered_apart_only_where_their_weights_are_the_tail(tmp_path):
    """One batch of 2561 to 4096 short rows is drawn by one launch, gathered and weighted by another; without weights there is
    no tail to take away, and those of more samples have a launch of their own behind draw and gather."""
    shapes = [(ob, k, w) for ob in (32, 1024, 1025) for k in (2049, 2560, 2561, 4096, 4097, 32_768) for w in (True, False)]
    out = recorded_hip.run(tmp_path, """
result = []
for obs_bytes, k, weights in %r:
    r = replay(50_000, obs_bytes)
    assert call("apex_replay_sample", r, 1, k, 0.4, memory(), memory(), memory(), memory() if weights else None, memory(),
                memory(), memory(), memory(), None) == 0
    result.append([x["kernel"] for x in launches()])
    assert call("apex_replay_destroy", r) == 0
""" % shapes)
    for (ob, k, weights), names in zip(shapes, out):
        apart = weights and 2560 < k <= 4096 and ob <= 1024
        assert "sample_kernel" in names[0] and len(names) == (2 if apart or weights and k > 4096 else 1), (ob, k, weights)
        assert any("finish_short" in n for n in names) == apart
        assert any("batch_weights" in n for n in names) == (weights and k > 4096)


def test_large_adds_of_the_shortest_rows_take_large_workgroups(tmp_path):
    """Adds of short rows in one launch: small workgroups for the rows' sake, large ones where the atomics of many
    transitions on the upper levels outweigh short rows."""
    shapes = [(16, 300), (16, 16_384), (16, 16_385), (16, 200_000), (16, 200_001), (64, 200_001), (65, 200_001), (256, 400_000)]
    out = recorded_hip.run(tmp_path, """
result = []
for obs_bytes, count in %r:
    r = replay(1 << 20, obs_bytes, filled=100)
    assert call("apex_replay_add", r, count, *[memory() for _ in range(5)], None, None) == 0
    result.append([[x["kernel"], x["grid"], x["block"]] for x in launches()])
""" % shapes)
    for (ob, count), found, threads in zip(shapes, out, (256, 256, 512, 512, 1024, 1024, 512, 512)):
        (kernel, grid, block), = found
        assert "add_rows_kernel" in kernel and (grid, block) == (-(-count // threads), threads), (ob, count)
