"""Host side of the library under several threads, on the CPU: libmgc.so runs
against a stand-in for the HIP runtime (hip_stub.cpp), in a process of its own."""
import os
import re
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.fixture(scope="module")
def on_stub(tmp_path_factory):
    """Runs a program text against libmgc.so (as `lib`) and the stand-in (as `hip`)."""
    import paper_2503_06322_amd as mgc
    path = mgc.library_path()
    if not os.path.exists(path):
        pytest.skip("libmgc.so not built")
    out = tmp_path_factory.mktemp("hip_stub")
    src = open(os.path.join(HERE, "hip_stub.cpp")).read()
    names = subprocess.run(["nm", "-D", "--undefined-only", path], capture_output=True, text=True, check=True).stdout
    wanted = set(re.findall(r"U (_*hip\w+)", names)) - set(re.findall(r"^\S.*?\b(_*hip\w+)\(", src, flags=re.M))
    (out / "rest.cpp").write_text("".join('extern "C" int %s() { return 0; }\n' % n for n in sorted(wanted)))
    soname = "libamdhip64.so.7"
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-pthread", "-Wl,-soname," + soname, "-o", str(out / soname),
                    os.path.join(HERE, "hip_stub.cpp"), str(out / "rest.cpp")], check=True)

    def run(program):
        head = "import ctypes, threading\nhip = ctypes.CDLL(%r)\nlib = ctypes.CDLL(%r)\n" % (soname, path)
        env = dict(os.environ, LD_LIBRARY_PATH=str(out), PYTHONPATH=ROOT)
        r = subprocess.run([sys.executable, "-c", head + program], capture_output=True, text=True, env=env, timeout=100)
        assert r.returncode == 0, r.stdout + r.stderr
    return run


OPEN = """
ctx = ctypes.c_void_p()
assert lib.mgc_create(0, ctypes.byref(ctx)) == 0
"""


def test_reads_of_two_threads_keep_apart(on_stub):
    """Each thread reads words of its own, waiting while the other's read is under way."""
    on_stub(OPEN + """
wrong = []
def reader(tag):
    words = (ctypes.c_uint64 * 128)(*[tag * 1000 + i for i in range(128)])
    got = (ctypes.c_uint64 * 128)()
    for k in range(100):
        ctypes.memset(got, 0, 1024)
        st = lib.mgc_read_prefix(ctx, words, ctypes.c_size_t(1024), got, None)
        if st != 0 or list(got) != list(words):
            wrong.append(tag)
threads = [threading.Thread(target=reader, args=(t,)) for t in range(1, 5)]
[t.start() for t in threads]
[t.join() for t in threads]
assert not wrong, "%d of 400 reads returned another thread's words" % len(wrong)
assert lib.mgc_destroy(ctx) == 0
""")


def test_reading_a_header_leaves_the_current_device(on_stub):
    """A program works on device 1 and looks at a stream that lies on device 0."""
    on_stub(OPEN + """
words = (ctypes.c_uint64 * 4)(1, 2, 3, 4)
got = (ctypes.c_uint64 * 4)()
hip.hipSetDevice(1)
assert lib.mgc_read_prefix(ctx, words, ctypes.c_size_t(32), got, None) == 0
dev = ctypes.c_int(-1)
hip.hipGetDevice(ctypes.byref(dev))
assert list(got) == [1, 2, 3, 4] and dev.value == 1, (list(got), dev.value)
# a refused read too
assert lib.mgc_read_prefix(ctx, words, ctypes.c_size_t(5000), got, None) == 1
hip.hipGetDevice(ctypes.byref(dev))
assert dev.value == 1
""")


def test_first_look_at_a_header_leaves_the_current_device(on_stub):
    """The same through the binding, where the look also creates the library's context."""
    on_stub("""
import contextlib, struct, types
import paper_2503_06322_amd as mgc
@contextlib.contextmanager
def device(d):
    before = ctypes.c_int()
    hip.hipGetDevice(ctypes.byref(before))
    hip.hipSetDevice(d)
    yield
    hip.hipSetDevice(before.value)
cuda = types.SimpleNamespace(device=device, current_stream=lambda d: types.SimpleNamespace(cuda_stream=0))
mgc._torch = lambda: types.SimpleNamespace(cuda=cuda)
buf = (ctypes.c_uint64 * 8)(5, 6, 7)
stream = types.SimpleNamespace(numel=lambda: 64, is_cuda=True, is_contiguous=lambda: True, element_size=lambda: 1,
                               device=types.SimpleNamespace(index=0), data_ptr=lambda: ctypes.addressof(buf))
hip.hipSetDevice(1)
for _ in range(2):
    assert struct.unpack("<3Q", mgc._prefix(stream, 24)) == (5, 6, 7)
    dev = ctypes.c_int(-1)
    hip.hipGetDevice(ctypes.byref(dev))
    assert dev.value == 1, dev.value
""")
