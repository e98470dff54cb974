"""Host code of the library against a stand-in runtime (no GPU): what a failed call leaves, and which kernels run."""
import subprocess

from tests import fake_device


def test_a_repeated_allocation_leaves_no_error(tmp_path):
    # one allocation fails for want of memory, its repetition succeeds: so does the call, whichever it was
    fake_device.run(tmp_path, """
def calls():
    ix = index(300)
    q = rows(20)
    for nq in (1, 20):
        apss.query(ix.handle, nq, q[0][:nq + 1], q[1][:2 * nq], q[2][:2 * nq], 0.5)
    ix.join(0.5)
    ix.close()

fake.fake_fail_mallocs(0, 0)
calls()
reached = 0
for k in range(fake.fake_mallocs()):
    fake.fake_fail_mallocs(k, 1)
    calls()
    reached += fake.fake_mallocs() > k  # (memory that is kept needs no call)
assert reached > 4
""")


# An index with postings: k_cutoff indexes every component, scans add up, and the deep lists hold `deep` entries in
# `units` wide units.
LISTS = """
deep, units = 600, 1 << 20
P64 = ctypes.POINTER(ctypes.c_int64)
arg = lambda args, k, t: ctypes.cast(args[k], ctypes.POINTER(t))[0]
at = lambda args, k: arg(args, k, P64)

@ctypes.CFUNCTYPE(None, ctypes.c_char_p, ctypes.POINTER(ctypes.c_void_p))
def hook(name, args):
    name = name.decode()
    if "k_cutoff" in name:
        rp, nidx = at(args, 0), at(args, 9)
        for r in range(arg(args, 3, ctypes.c_int64)):
            nidx[r] = rp[r + 1] - rp[r]
    elif "k_scan_chunk" in name:
        data, n, total = at(args, 0), arg(args, 1, ctypes.c_int64), 0
        assert n <= 2048
        for k in range(n):
            data[k], total = total, total + data[k]
        at(args, 2)[0] = total
    elif "k_count_deep" in name:
        at(args, 2)[0] = deep
    elif "k_unit_countsILb1E" in name:
        at(args, 2)[0] = units

fake.fake_hook(hook)

def joined(ix):
    launches()
    ix.join(0.5)
    return launches()

ran = lambda kernel, names: any(kernel in k for k in names)
"""


def test_an_index_without_room_for_pair_lists_is_built_without(tmp_path):
    # each allocation of a build fails in turn, for good: the index's own end the build with APSS_ENOMEM, those of the
    # list-pair tables alone leave an index whose joins take the accumulating kernel
    fake_device.run(tmp_path, LISTS + """
import os

def outcome(k):  # of a build, in a process of its own, whose k-th allocation and its repetition fail
    fake.fake_fail_mallocs(k, 2)
    try:
        ix = index(600)
    except apss.ApssError as e:
        assert e.code == apss.APSS_ENOMEM
        return 1
    reached = fake.fake_mallocs() > k
    fake.fake_fail_mallocs(0, 0)
    names = joined(ix)
    assert ran("k_pairs_wide", names) != reached and ran("k_join", names) == reached
    return 2 if reached else 3

got = []
while 3 not in got:
    if not (pid := os.fork()):
        os._exit(outcome(len(got)))
    got.append(os.waitstatus_to_exitcode(os.waitpid(pid, 0)[1]))
    assert got[-1] in (1, 2, 3) and len(got) < 30
assert got.count(2) == 2 and got.count(1) >= 3, got
""")


def test_more_units_than_the_pair_kernels_count(tmp_path):
    # lists so long that their pairs make 2^31 work units (22 million rows over few dimensions): the accumulating kernel
    fake_device.run(tmp_path, LISTS + """
for units in (2**31, 9 * 2**31):
    names = joined(index(600))
    assert ran("k_join", names) and not ran("k_pairs", names)
""")


def test_a_batch_that_overflows_is_not_counted_before(tmp_path):
    # the sketch tests come before the exact count, which is as long; a flagged batch is made again by the other kernel
    fake_device.run(tmp_path, LISTS + """
o = apss.default_opts()
o.reserved[0] = 0x50414952  # sketches whatever the cost rule says
ix = apss.Index(apss.build_index(600, 64, *rows(600), 0.5, o), 600, 64)
flags = [1]

@ctypes.CFUNCTYPE(None, ctypes.c_char_p, ctypes.POINTER(ctypes.c_void_p))
def finish(name, args):
    if b"k_finish" in name:
        host = ctypes.cast(args[0] + 80, ctypes.POINTER(P64))[0]  # FinishArgs.host
        host[7] = flags.pop() if flags else 0  # C_OVERFLOW

fake.fake_hook(finish)
launches()
q = rows(40)
apss.query(ix.handle, 40, *q, 0.5)
names = [k for k in launches() if any(x in k for x in ("k_query_screen", "k_decide", "k_count", "k_join", "k_finish"))]
order = ["k_query_screen", "k_decide", "k_count", "k_finish", "k_join", "k_finish"]
assert len(names) == len(order) and all(o in k for o, k in zip(order, names)), names
""")


def test_negative_capacities_are_too_small(tmp_path):
    fake_device.run(tmp_path, """
ix, q, cnt = index(300), rows(20), ctypes.c_int64(7)
lib = apss.load()
for n in (300, 0):
    ix = index(n) if n else apss.Index(apss.build_index(0, 64, np.zeros(1, np.int64), q[1], q[2], 0.5, apss.default_opts()), 0, 64)
    assert lib.apss_join_device(ix.handle, 0.5, None, None, None, -1, ctypes.byref(cnt)) == apss.APSS_ERANGE
    assert cnt.value == 0 and "capacity -1" in apss.last_error()
    for nq in (1, 20):
        assert lib.apss_query_device(ix.handle, nq, *[x.ctypes.data for x in q], 0, None, 0.5, None, None, None, -5,
                                     ctypes.byref(cnt)) == apss.APSS_ERANGE
    assert lib.apss_join_device(ix.handle, 0.5, None, None, None, 0, ctypes.byref(cnt)) == apss.APSS_OK
""")


def test_query_rows_without_components_arrays(tmp_path):
    # NULL arrays of a batch that has components: refused, small batches (which are packed on the host) and large ones
    fake_device.run(tmp_path, """
ix, p = index(300), apss.Pairs()
lib = apss.load()
for nq in (1, 20, 20000):
    q = rows(nq)
    rp, c, v = [x.ctypes.data for x in q]
    for args in ((rp, None, v), (rp, c, None), (rp, None, None)):
        for device in (0, 1):
            assert lib.apss_query(ix.handle, nq, *args, device, None, 0.5, ctypes.byref(p)) == apss.APSS_EINVAL
    assert lib.apss_query(ix.handle, nq, rp, c, v, 0, None, 0.5, ctypes.byref(p)) == apss.APSS_OK
empty = np.zeros(4, np.int64)
assert lib.apss_query(ix.handle, 3, empty.ctypes.data, None, None, 0, None, 0.5, ctypes.byref(p)) == apss.APSS_OK
""")


def test_a_query_that_fails_leaves_nothing_to_the_next_call(tmp_path):
    # a query whose rows were staged, and which then failed before its kernels: the next call clears its own counters
    fake_device.run(tmp_path, """
ix, q = index(300), rows(20)
cnt = ctypes.c_int64()
ix.join(0.5)
for call in (lambda: ix.join(0.5), lambda: apss.load().apss_join_device(ix.handle, 0.5, None, None, None, 0, ctypes.byref(cnt))):
    launches()
    call()
    want = launches()
    for nq in (1, 20):
        for event in (0, 1):
            fake.fake_fail_events(event, 1)
            try:
                apss.query(ix.handle, nq, q[0][:nq + 1], q[1][:2 * nq], q[2][:2 * nq], 0.5)
                assert False
            except apss.ApssError as e:
                assert e.code == apss.APSS_EDEVICE
            fake.fake_fail_events(0, 0)
            fake.hipGetLastError()
            launches()
            call()
            assert launches() == want
""")


def test_kept_memory_goes_back_when_asked(tmp_path):
    fake_device.run(tmp_path, """
assert apss.release_memory() == 0
for _ in range(2):
    a, b = index(300), index(5000)
    a.close()
    c = index(300)  # (from what the first one left)
    c.join(0.5)
    b.close()
    c.close()
    assert fake.fake_live() > 0  # kept for the next index
    assert apss.release_memory() >= 3 << 20
    assert fake.fake_live() == 0 and apss.release_memory() == 0
""")


def test_ending_an_index_needs_no_host_memory(tmp_path):
    # operator new fails in apss_index_free, at each of its calls in turn: the chunks are freed in place of kept
    src = tmp_path / "new.cpp"
    src.write_text("""
#include <cstdlib>
#include <new>
static long calls, from = -1;
extern "C" void fake_fail_news(long k) { calls = 0; from = k; }
extern "C" long fake_news() { return calls; }
void* operator new(std::size_t n) {
  if (from >= 0 && calls++ >= from) throw std::bad_alloc();
  return std::malloc(n);
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, std::size_t) noexcept { std::free(p); }
""")
    lib = tmp_path / "new.so"
    subprocess.run(["g++", "-shared", "-fPIC", "-O1", str(src), "-o", str(lib)], check=True)
    fake_device.run(tmp_path, """
for k in range(3):
    ixs = [index(n) for n in (300, 5000, 70000)]
    news.fake_fail_news(ctypes.c_long(k))
    for ix in ixs:
        ix.close()
    used = news.fake_news()
    news.fake_fail_news(ctypes.c_long(-1))
    assert used > 0 or k > 0
    apss.release_memory()
    assert fake.fake_live() == 0
""", before="news = ctypes.CDLL(%r, ctypes.RTLD_GLOBAL)\n" % str(lib))


def test_the_environment_counts_when_an_index_is_built(tmp_path):
    # an index keeps its kernels when the variables change after its build
    fake_device.run(tmp_path, """
import os
q = rows(3)

def kernels(ix):
    launches()
    apss.query(ix.handle, 3, *q, 0.5)
    return [k for k in launches() if "k_few" in k or "k_join" in k]

default = index(300)
assert "k_few" in kernels(default)[0]
for name, value in (("APSS_VARIANT", "0"), ("APSS_RANGE_ROWS", "4096"), ("APSS_RANGE_GROUP", "2")):
    os.environ[name] = value
    assert len(kernels(default)) == 1 and "k_few" in kernels(default)[0]
    named = index(300)
    assert "k_join" in kernels(named)[0]
    del os.environ[name]
    assert "k_join" in kernels(named)[0]
""")
