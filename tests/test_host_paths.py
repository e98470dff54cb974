"""Host code of the library against a stand-in runtime (no GPU): what a failed call leaves, and which kernels run."""
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
