"""CPU-only checks of the boundary: the library loads and exports what the header declares."""
import ctypes as C
import os
import re

from conftest import ROOT

HEADER = os.path.join(ROOT, "include", "apex_replay.h")


def declared_functions():
    text = open(HEADER).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(?:int|size_t)\s+(apex_\w+)\s*\(", text)))


def test_header_declares_the_replay_verbs():
    names = declared_functions()
    for verb in ("apex_replay_create", "apex_nstep_priorities", "apex_replay_add", "apex_replay_sample",
                 "apex_replay_update_priorities", "apex_replay_evict"):
        assert verb in names


def test_library_exports_every_declared_symbol():
    from paper_1803_00933_amd import apex
    for name in declared_functions():
        assert hasattr(apex.lib, name), name
    assert sorted(apex.EXPORTS) == declared_functions()


def test_struct_sizes_match_the_header():
    from paper_1803_00933_amd import apex
    assert C.sizeof(apex.Config) == 48
    assert C.sizeof(apex.Stats) == 48
    assert C.sizeof(apex.Layout) == 4 * 8 + 8 + 2 * 8 * apex.TREE_MAX_LEVELS
    text = open(HEADER).read()
    assert "#define APEX_MAX_SAMPLES_PER_CALL %du" % apex.MAX_SAMPLES_PER_CALL in text
    assert "#define APEX_MAX_BATCHES_PER_CALL %du" % apex.MAX_BATCHES_PER_CALL in text
    assert "#define APEX_TREE_MAX_LEVELS %du" % apex.TREE_MAX_LEVELS in text


def test_workspace_sizes_and_argument_checks_need_no_gpu():
    from paper_1803_00933_amd import apex
    cfg = apex.Config(2_000_000, 1 << 21, 28224, 4, 0.6, 1e-6, 24, 0, 0)
    rc, storage, tree, scratch = apex.workspace_bytes(cfg)
    assert rc == apex.OK
    P = 1 << 21
    assert storage == P * 28224 + P * 4 * 3
    assert tree == 2 * 8 * (P + P // 64 + P // 4096)      # three levels: 2^21, 2^15, 2^9 nodes; two copies
    assert scratch >= P * 4
    for bad in (apex.Config(0, 8, 4, 4, 0.6, 0, 24, 0, 0), apex.Config(9, 8, 4, 4, 0.6, 0, 24, 0, 0),
                apex.Config(8, 8, 0, 4, 0.6, 0, 24, 0, 0), apex.Config(8, 8, 4, 4, 1.5, 0, 24, 0, 0),
                apex.Config(8, 8, 4, 4, 0.6, -1.0, 24, 0, 0), apex.Config(8, 8, 4, 4, 0.6, 0, 33, 0, 0),
                apex.Config(8, 8, 4, 4, float("nan"), 0, 24, 0, 0)):
        assert apex.workspace_bytes(bad)[0] == apex.ERR_INVALID_ARG
    assert apex.lib.apex_replay_destroy(None) == apex.ERR_INVALID_ARG
    assert apex.lib.apex_nstep_priorities(0, 1, 1, 1, *([None] * 5), 0.6, 0.0, 24, 0, *([None] * 5)) == apex.ERR_INVALID_ARG


def test_synthetic_observation_bytes_agree_between_numpy_and_torch():
    import numpy as np
    import torch
    from paper_1803_00933_amd import synth
    a = synth.obs_rows(7, (1 << 40) + 3, 11, 64)
    b = synth.obs_rows_torch(7, (1 << 40) + 3, 11, 64, "cpu").numpy()
    assert np.array_equal(a, b)
    assert len(np.unique(a)) > 200                                  # looks like uniform bytes
    assert np.array_equal(synth.obs_rows(7, (1 << 40) + 5, 2, 64), a[2:4])   # a pure function of the key


def test_rows_for_scattered_keys_are_the_rows_of_those_keys():
    import numpy as np
    from paper_1803_00933_amd import synth
    keys = np.array([5, (1 << 40) + 3, 5, 0, (1 << 63) + 17, 123456789], dtype=np.uint64)
    got = synth.obs_rows_for_keys_torch(7, keys, 128, "cpu").numpy()
    for i, k in enumerate(keys):
        assert np.array_equal(got[i], synth.obs_rows(7, int(k), 1, 128)[0])
    got = synth.frame_rows_for_keys_torch(7, keys, 128, "cpu").numpy()
    for i, k in enumerate(keys):
        assert np.array_equal(got[i], synth.frame_rows(7, int(k), 1, 128)[0])
    assert np.array_equal(synth.frame_rows_torch(7, 40, 9, 256, "cpu").numpy(), synth.frame_rows(7, 40, 9, 256))


def test_null_handles_are_refused_without_a_gpu():
    from paper_1803_00933_amd import apex
    lib, bad = apex.lib, apex.ERR_INVALID_ARG
    assert lib.apex_replay_sample_noalloc(None, 1, 8, 0.4, *([None] * 9)) == bad
    assert lib.apex_replay_sample(None, 1, 8, 0.4, *([None] * 9)) == bad
    assert lib.apex_replay_update_priorities(None, 0, None, None, None) == bad
    assert lib.apex_replay_evict(None, None, None) == bad
    assert lib.apex_pipeline_steps(None, 1, 0.4, None, None, None) == bad
    assert lib.apex_pe_evict_enqueue(None, 1, None, None, None) == bad
    assert lib.apex_pe_add_round(None, 1, 1, 1, 1, *([None] * 8)) == bad
    assert lib.apex_pe_sample_update(None, 8, 0.4, *([None] * 10)) == bad
    assert lib.apex_pe_destroy(None) == bad and lib.apex_pipeline_destroy(None) == bad
    pe = apex.PeConfig(10, 8, 16, 4, 0.6, -0.4, 1e-6, 24)              # max_slots < capacity
    a = C.c_size_t(0)
    assert lib.apex_pe_workspace_bytes(C.byref(pe), C.byref(a), None, None) == bad
    pe = apex.PeConfig(1_000_000, 1 << 20, 256, 32, 0.6, -0.4, 1e-6, 24)
    assert lib.apex_pe_workspace_bytes(C.byref(pe), C.byref(a), None, None) == apex.OK and a.value >= (1 << 20) * 256
    assert int(lib.apex_codec_row_bytes(28224)) == 28736 and int(lib.apex_codec_row_bytes(100)) == 0


def test_uniforms_of_an_eviction_cover_what_the_library_addresses():
    """Whatever number of evictions turns out to be due, the library is handed rounds * e words or the call is refused:
    a tensor that is long enough as it is, a shorter one with its words repeated, one too short for the first round not."""
    import pytest
    import torch
    from paper_1803_00933_amd import apex
    rnd = torch.arange(12).view(3, 4)
    for rounds, e in ((3, 4), (3, 0), (2, 6), (1, 12), (0, 50)):
        assert apex.eviction_uniforms(rnd, rounds, e) is rnd
    for rounds, e in ((3, 5), (3, 12), (7, 11)):
        whole = apex.eviction_uniforms(rnd, rounds, e)
        assert whole.is_contiguous() and whole.numel() >= rounds * e
        assert torch.equal(whole, torch.arange(whole.numel()) % 12)
    for rounds, e in ((1, 13), (3, 100)):
        with pytest.raises(ValueError):
            apex.eviction_uniforms(rnd, rounds, e)


def test_binding_refuses_what_it_cannot_address():
    """The calls marshalled by the extension: the library's status for a missing handle, and errors for tensors that have
    no device address to give, for numbers that are none, and for a wrong count of arguments."""
    import pytest
    import torch
    from paper_1803_00933_amd import apex
    call, bad = apex._call, apex.ERR_INVALID_ARG

    class stream:
        cuda_stream = 0

    assert call.update_priorities(None, 0, None, None, stream) == bad
    assert call.evict(None, stream) == (bad, 0) and call.pipeline_add_end(None, 1) == (bad, 0, 0)
    assert call.pipeline_steps(None, 1, 0.4, None, None) == (bad, 0) and call.pipeline_fork(None, stream) == bad
    for t in (torch.zeros(4), torch.zeros((4, 4)).t()):
        with pytest.raises(AssertionError):
            call.update_priorities(None, 1, t, None, stream)
    with pytest.raises(AttributeError):
        call.update_priorities(None, 1, 4096, None, stream)             # a bare address is no tensor
    for args in ((None, 1.0, None, None, stream), (None, "1", None, None, stream), ("h", 1, None, None, stream)):
        with pytest.raises(TypeError):
            call.update_priorities(*args)
    with pytest.raises(TypeError):
        call.update_priorities(None, 0, None, None)
    with pytest.raises(TypeError):
        call.pipeline_steps(None, 1, "0.4", None, None)
    with pytest.raises(AttributeError):
        call.evict(None, 7)                                             # no stream


def test_binding_takes_every_number_that_ctypes_takes():
    """Counts and exponents as numpy has them, or anything else with an index or a float value, ctypes' own scalars, objects
    that name their argument, and streams whose handle is none of Python's integers."""
    import numpy as np
    import pytest
    from paper_1803_00933_amd import apex
    call, bad = apex._call, apex.ERR_INVALID_ARG

    class Named:
        def __init__(self, value):
            self._as_parameter_ = value

    class Indexed:
        def __index__(self):
            return 3

    class Stream:
        def __init__(self, handle):
            self.cuda_stream = handle

    for number in (3, True, np.int64(3), np.uint32(3), np.uint8(3), C.c_uint64(3), Named(3), Named(C.c_uint64(3)), Indexed(), -1):
        apex.lib.apex_replay_update_priorities(None, number, None, None, None)          # ctypes takes it
        assert call.update_priorities(None, number, None, None, Stream(0)) == bad, number
    for number in (0.4, 1, np.float32(0.4), np.float64(0.4), np.int64(1), C.c_float(0.4), Named(0.4), Indexed()):
        assert call.pipeline_steps(None, 1, number, None, None) == (bad, 0), number
    for handle in (0, None, np.int64(0), C.c_void_p(), C.c_void_p(0), Named(0)):
        assert call.evict(None, Stream(handle)) == (bad, 0), handle
    for number in (3.0, np.float32(3), "3", None, Named("3"), C.c_float(3)):
        with pytest.raises(TypeError):
            call.update_priorities(None, number, None, None, Stream(0))
    for number in ("0.4", None, Named(None), C.c_char(b"0")):
        with pytest.raises(TypeError):
            call.pipeline_steps(None, 1, number, None, None)


def test_binding_survives_an_exception_out_of_the_library(tmp_path):
    """The interpreter's lock is given up for a call and taken back however the call ends: an exception becomes Python's."""
    import subprocess
    import sys
    from paper_1803_00933_amd import apex
    src, so = str(tmp_path / "throwing.cpp"), str(tmp_path / "throwing.so")
    with open(src, "w") as f:
        f.write("#include <new>\n" + "\n".join('extern "C" int %s() { throw std::bad_alloc(); }' % n for n in apex.EXPORTS))
    subprocess.check_call(["g++", "-O1", "-shared", "-fPIC", "-o", so, src])
    code = """
import sys, threading, torch
from paper_1803_00933_amd import apex
apex._call.load(sys.argv[1], apex._ptr, apex._plain, None, None)
class stream: cuda_stream = 0
other, stop = [0], threading.Event()
def count():
    while not stop.is_set(): other[0] += 1
t = threading.Thread(target=count)
t.start()
for i in range(1000):
    try:
        apex._call.evict(None, stream)
    except RuntimeError as e:
        assert "bad_alloc" in str(e)
    else:
        raise SystemExit("no exception")
stop.set(); t.join()
print("passed", other[0] > 0)
"""
    r = subprocess.run([sys.executable, "-c", code, so], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "passed True" in r.stdout, (r.returncode, r.stderr[-2000:])
