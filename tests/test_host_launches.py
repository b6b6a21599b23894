"""The library's host side on a recording stand-in of the HIP runtime (host_stub.py):
what it launches, refuses and sizes, at sizes and failures that need no GPU."""
import host_stub


def test_appended_rows_beyond_32_bits(tmp_path):
    """Steps that append batch x n_new rows of `hidden` columns, 2^31 and 2^32 values of
    them among the sizes: the launch that writes the rows as fragment planes has eight columns
    a thread, no more threads than a grid holds, and none missing."""
    host_stub.run('''
for fuse in (0, 5):
    m = h.Model(h.config(4096, 32, 12288, vocab=4096, fuse=fuse))
    for batch, n_new in ((1, 1), (3, 7), (64, 8191), (64, 8192), (64, 16448)):
        st = m.step(batch, 17000, n_new, 1 << 40)
        assert st == 0, (batch, n_new, st)
        grids = [r for r in h.log() if r[0] == "launch" and "sum_parts_planes" in r[1]]
        assert len(grids) == 1
        threads = int(grids[0][2]) * int(grids[0][5])
        assert batch * n_new * 4096 // 8 <= threads < 2**32, (fuse, batch, n_new, threads)
        assert grids[0][3:5] == ["1", "1"]
''', tmp_path)


def test_a_workspace_serves_any_number_of_appended_rows(tmp_path):
    """A program allocates once for max_new and appends what each cycle accepted: no step or
    training forward of fewer rows is refused, one byte less than a step's own need is."""
    host_stub.run('''
def need(call, most):
    """Least bytes that `call` accepts, by bisection."""
    lo, hi = 0, most
    while lo < hi:
        mid = (lo + hi) // 2
        lo, hi = (mid + 1, hi) if call(mid) == -2 else (lo, mid)
    h.log()
    return lo

shapes = {s: h.config(*h.SHAPES[s]) for s in h.SHAPES}
shapes["plain"] = h.config(4096, 32, 12288, fuse=0)
shapes["f32"] = h.config(256, 4, 1024, vocab=4096, fuse=0, dtype=0, nkv=2, head_dim=64)
for name, cfg in shapes.items():
    m = h.Model(cfg)
    for batch in list(range(1, 13)) + [16, 24, 33, 64]:
        for most in (1, 5, 8, 15, 16, 64):
            ws, tws = m.ws(batch, 2048, most), m.train_ws(batch, 2048, most)
            for n in range(most + 1):
                assert m.step(batch, 2048, n, ws) == 0, (name, batch, most, n)
                assert m.train(batch, 2048, n, tws) == 0, (name, batch, most, n)
            h.log()
    for batch, n in ((1, 0), (1, 5), (2, 9), (9, 16)):
        own = need(lambda b: m.step(batch, 2048, n, b), m.ws(batch, 2048, n))
        assert own > 0 and m.step(batch, 2048, n, own - 1) == -2
''', tmp_path)


ROLLOUT = '''
PERSIST = "head_persist"

def step(m, batch=1, stream=0, branch=1):
    """The stream calls of one step's rollout: waits, the persistent launch, records."""
    h.log()
    assert m.step(batch, 2048, 0, 1 << 40, branch=branch, stream=stream) == 0
    return [(r[0] if r[0] != "launch" else PERSIST, int(r[-1])) for r in h.log()
            if r[0] in ("wait", "record") or PERSIST in r[1]]

m = h.Model(h.config(*h.SHAPES["8b"]))
def ordered(s): return [("wait", s), (PERSIST, s), ("record", s)]
'''


def test_persistent_rollouts_wait_for_the_last_one(tmp_path):
    """Whatever its stream: hipStreamPerThread (2) is another stream in another thread, and a
    handle may be that of a new stream."""
    host_stub.run(ROLLOUT + '''
assert step(m) == [(PERSIST, 0), ("record", 0)]
for s in (0, 77, 77, 2, 2, 0):
    assert step(m, stream=s) == ordered(s), s
assert step(m, batch=8, branch=3, stream=5) == ordered(5)
''', tmp_path)


def test_rollouts_that_cannot_be_ordered_go_launch_by_launch(tmp_path):
    host_stub.run(ROLLOUT + '''
def loops(**kw):
    return step(m, **kw) == [] and m.paths() == 0

h.stub.stub_fail(b"hipEventCreateWithFlags", 1)
assert loops()
assert step(m) == [(PERSIST, 0), ("record", 0)] and m.paths() == 1
h.stub.stub_fail(b"hipStreamWaitEvent", 1)
assert loops(stream=9)
assert step(m, stream=9) == ordered(9)
h.stub.stub_fail(b"hipGetDevice", 1)
assert loops()
h.stub.stub_fail(b"hipEventRecord", 1)   # a launch that nothing can wait for any more
assert step(m, stream=9) == [("wait", 9), (PERSIST, 9)]
assert loops() and loops(stream=9) and loops(batch=3, branch=2)
''', tmp_path)


def test_captured_rollouts(tmp_path):
    """A graph's replays are not ordered: only up to four rows with one candidate a position
    are captured as the persistent launch; nothing waits or records during a capture."""
    host_stub.run(ROLLOUT + '''
assert step(m, batch=5, branch=2) == [(PERSIST, 0), ("record", 0)]
h.stub.stub_capture(31, 1)
for batch, branch in ((1, 1), (4, 1)):
    assert step(m, batch=batch, branch=branch, stream=31) == [(PERSIST, 31)] and m.paths() == 1
for batch, branch in ((5, 1), (8, 1), (1, 2), (4, 8)):
    assert step(m, batch=batch, branch=branch, stream=31) == [] and m.paths() == 0
h.stub.stub_capture(31, 0)
assert step(m, batch=8, branch=8, stream=31) == ordered(31)
''', tmp_path)
