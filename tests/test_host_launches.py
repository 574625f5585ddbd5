"""What the library asks of the HIP runtime, call by call, without a GPU (host_hip.py)."""
import pytest

import host_hip


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return host_hip.build(str(tmp_path_factory.mktemp("fake_hip")))


# Pointers of the parameters are sent by the first step that reads them from the tables on the GPU.  A send that is recorded into a
# graph writes nothing until the graph is replayed, and then in every replay: steps outside of it cannot rely on what is there.
def test_pointer_tables_are_sent_where_a_recorded_send_may_not_have_run(lib):
    out = host_hip.run(lib, r"""
o = Opt([(96, 128), (40,)], 128, freq=100)
def sends(t, where, capturing=0):
    reset(capturing=capturing)
    assert o.step(t, where) == 0
    return len(launches("pointer_table_kernel"))
print(sends(100, 1), sends(101, 1), sends(102, 3))      # a refresh; steps in one kernel, which bring their pointers along
print(sends(200, 3, 1))                                 # a refresh, recorded
print(sends(300, 3))                                    # an eager one before any replay
print(sends(400, 3, 1), sends(500, 3))                  # recorded again; an eager one that a replay may have come before
print(sends(600, 5), sends(700, 5))
""")
    assert out[:5] == ["1 0 0", "1", "1", "1 1", "1 1"], out


def test_pointers_that_fit_a_launch_travel_with_it(lib):
    out = host_hip.run(lib, r"""
for count in (224, 225):
    o = Opt([(24, 20), (7,)] * (count // 2) + [(9,)] * (count % 2), 64)
    assert o.step(1, 1) == 0
    reset()
    assert o.step(2, 3) == 0
    print(len(launches("pointer_table_kernel")), len(launches()))
""")
    assert out[:2] == ["0 1", "1 2"], out


def test_a_recorded_step_brings_its_pointers(lib):
    """Replays work on the tensors that the step was recorded with, whichever steps come between them."""
    out = host_hip.run(lib, r"""
o = Opt([(300, 128)], 256, freq=100)
for t, where, capturing in ((0, 1, 0), (1, 1, 0), (2, 1, 1), (3, 3, 0), (4, 3, 0)):
    reset(capturing=capturing)
    assert o.step(t, where) == 0
    print(len(launches("pointer_table_kernel")))
""")
    assert out[:5] == ["1", "0", "1", "1", "1"], out


# Helper streams are forked off the caller's stream and joined to it.  Whatever fails in between, and wherever host memory runs out, the
# caller's stream waits for what is under way: memory that the caller frees after the error is not in use.  (A failing record or
# wait cannot be made up for.)
@pytest.mark.parametrize("what,call", [
    # small blocks beside the stages of large ones
    ("step", "o = Opt([(2124, 2048)] + [(96, 128)] * 40, 1024); o.step(0)\ncall = lambda: o.step(1)"),
    # band reductions on three streams, small roots on another
    ("refresh", "o = Opt([(160, 200)] * 40 + [(96, 128)], 256, freq=1); o.step(0)\ncall = lambda: o.step(1)"),
    # the Jacobi solver (no rational sum for this exponent)
    ("jacobi", """
ws = L.shampoo_root_inverse_workspace_bytes(130, 5)
call = lambda: L.shampoo_root_inverse(ctypes.c_void_p(1 << 36), 130, 5, 1e-12, 1.0, ctypes.c_void_p(1 << 37), None, None, ctypes.c_void_p(1 << 40), ws,
                                      ctypes.c_void_p(STREAM))
"""),
], ids=["step", "refresh", "jacobi"])
def test_a_call_that_fails_leaves_nothing_beside_the_callers_stream(lib, what, call):
    out = host_hip.run(lib, "reset()\n" + call + r"""
reset()
assert call() == 0 and unjoined() == []
assert any(e.stream not in (None, STREAM) for e in launches())       # there is something to join
bad, n, t = {"code": 0, "unjoined": 0}, 0, 1
def again():
    global t
    t += 1
    return call() if WHAT == "jacobi" else o.step(t)
for failed, rc in failing(again):
    n += 1
    bad["code"] += rc != -6
    bad["unjoined"] += failed not in "RW" and len(unjoined()) > 0
for rc in out_of_memory(again):
    n += 1
    bad["code"] += rc not in (0, -6)        # 0: a sort that did without its buffer
    bad["unjoined"] += len(unjoined()) > 0
print(n > 20, bad)
""".replace("WHAT", repr(what)))
    assert out[0] == "True {'code': 0, 'unjoined': 0}", out


@pytest.mark.parametrize("timing", [0, 1])
def test_a_first_step_that_runs_out_of_host_memory_can_be_taken_again(lib, timing):
    """Wherever the memory runs out: an error code, and the same call succeeds afterwards with what it sends to the GPU complete."""
    out = host_hip.run(lib, r"""
def fresh():
    global o
    reset()
    o = Opt([(300, 128), (40,), (20, 30, 9)], 256)
    o.timing(TIMING)
def first(k):
    reset(alloc_fail=k)
    fake.fake_count_allocations(1)
    rc = o.step(0)
    fake.fake_count_allocations(0)
    return rc, fake.fake_allocations()
fresh()
rc, allocations = first(-1)
want = [(e.name, e.a) for e in launches()]
assert rc == 0 and allocations > 5
bad = 0
for k in range(allocations):
    fresh()
    rc, _ = first(k)
    assert rc in (0, -6)
    if rc == 0:
        continue
    rc, _ = first(-1)
    got = [(e.name, e.a) for e in launches()]
    # the tables may have gone before the memory ran out
    bad += rc != 0 or [x for x in got if b"pointer_table" not in x[0]] != [x for x in want if b"pointer_table" not in x[0]]
print("ok", bad)
""".replace("TIMING", str(timing)))
    assert out[0] == "ok 0", out


def test_a_state_query_completes_the_one_factor_that_it_returns(lib):
    """Upper triangles (small blocks) and tiles above the diagonal are written on request: of one matrix, not of its bucket."""
    out = host_hip.run(lib, r"""
for shapes, block, n in (([(96, 128)] * 50, 128, 128), ([(2048, 2048)] * 3, 1024, 1024)):
    o = Opt(shapes, block, grad_dtype=B.GRAD_BF16)
    for t in (0, 1):
        assert o.step(t) == 0
    for which in (B.GET_L, B.GET_R):
        dim = 96 if n == 128 and which == B.GET_L else n
        reset()
        assert o.get(1, 0, which, dim * dim * 4) == 0
        print([e.a for e in launches("mirror")], (-(-dim // 32)) ** 2)
    reset()
    assert o.get(1, 0, B.GET_LINV, (96 if n == 128 else n) ** 2 * 4) == 0
    print(len(launches()))
""")
    assert out[:6] == ["[16] 9", "[16] 16", "0", "[1024] 1024", "[1024] 1024", "0"], out


def test_upper_tiles_stay_marked(lib):
    """A replay of a step that leaves them out may come behind any other: once one has been enqueued they are always completed."""
    out = host_hip.run(lib, r"""
o = Opt([(264, 264)], 264, grad_dtype=B.GRAD_BF16)
def mirrors():
    reset()
    assert o.get(0, 0, B.GET_L, 264 * 264 * 4) == 0
    return len(launches("mirror"))
assert o.step(1, skew=2) == 0
print(mirrors())                       # unaligned gradients: that update writes all of the factor
assert o.step(2) == 0
print(mirrors())
assert o.step(3, skew=2) == 0
print(mirrors())
""")
    assert out[:3] == ["0", "1", "1"], out


@pytest.mark.parametrize("grad", ["GRAD_F32", "GRAD_BF16"])
def test_a_stage_of_a_step_is_one_interval(lib, grad):
    """Time per interval is time per step for parameters that are worked on together, as the benchmark takes it to be."""
    out = host_hip.run(lib, r"""
o = Opt([(300, 520), (40,)], 264, grad_dtype=B.GRAD)
o.timing(1)
for t in range(1, 4):
    assert o.step(t) == 0
o.timing(0)
for stage in (0, 1, 3, 4, 5, 7):
    ms, n = ctypes.c_double(), i64()
    assert L.shampoo_get_timing(o.handle, stage, ctypes.byref(ms), ctypes.byref(n)) == 0
    print(n.value)
""".replace("B.GRAD", "B." + grad))
    assert out[:6] == ["3"] * 6, out


@pytest.mark.parametrize("shapes", ["[(2124, 2048)] + [(96, 128)] * 40", "[(160, 200)] * 40 + [(96, 128)]", "[(40, 150, 9)]"])
def test_helper_streams_are_there_before_the_first_step(lib, shapes):
    """Neither a step nor a refresh makes streams, and one that is recorded first uses them like any other."""
    out = host_hip.run(lib, r"""
def run(capturing):
    reset()
    o = Opt(SHAPES, 1024, freq=2)
    seen = []
    for t in (0, 1):
        reset(capturing=capturing)
        assert o.step(t) == 0
        assert not [e for e in entries() if e.what in b"SE"], t
        seen.append(sorted((e.name, e.a, e.stream != STREAM) for e in launches() if b"pointer_table" not in e.name))
    return seen
a, b = run(0), run(1)
print(a == b, any(x[2] for step in a for x in step))
""".replace("SHAPES", shapes))
    assert out[0] == "True True", out


def test_roots_of_a_refresh_take_equal_passes(lib):
    """One pass over up to a matrix of 1024 for every CU, then two of the same size, each on three streams."""
    out = host_hip.run(lib, r"""
for count in (96, 128, 129, 200):
    o = Opt([(1024, 1024)] * count, 1024, freq=1)
    reset()
    assert o.step(1) == 0
    sides = [e.a for e in launches("band_alone")]
    print(len(sides), max(sides) - min(sides) <= 8, sum(sides) >= 2 * count)
""")
    assert out[:4] == ["3 True True", "3 True True", "6 True True", "6 True True"], out


@pytest.mark.parametrize("p,launches", [(1, 1), (2, 2), (4, 3), (8, 4)])
def test_products_of_a_newton_iteration(lib, p, launches):
    """X T goes along with the first of the others, whose squares and last product need one another."""
    out = host_hip.run(lib, r"""
ws = L.shampoo_root_inverse_newton_workspace_bytes(129, 3)
def call(iterations):
    reset()
    assert L.shampoo_root_inverse_newton(ctypes.c_void_p(1 << 36), 129, 3, ctypes.c_float(1e-6), P, ctypes.c_float(1e-6), iterations, ctypes.c_void_p(1 << 37), None,
                                         None, ctypes.c_void_p(1 << 40), ws, ctypes.c_void_p(STREAM)) == 0
    return len(launches("gemm_mfma_kernel"))
print(call(1), call(7))
""".replace("P,", "%d," % p, 1))
    assert out[0] == "%d %d" % (launches, 7 * launches), out


@pytest.mark.parametrize("n", [1, 40, 128])
def test_a_small_newton_iteration_is_one_launch(lib, n):
    """Whatever the cap: the arithmetic of a matrix does not change with the number of iterations that a call allows."""
    out = host_hip.run(lib, r"""
ws = L.shampoo_root_inverse_newton_workspace_bytes(N, 3)
for cap in (1, 7, 8, 1000):
    reset()
    assert L.shampoo_root_inverse_newton(ctypes.c_void_p(1 << 36), N, 3, ctypes.c_float(1e-6), 4, ctypes.c_float(1e-6), cap, ctypes.c_void_p(1 << 37), None,
                                         None, ctypes.c_void_p(1 << 40), ws, ctypes.c_void_p(STREAM)) == 0
    print(len(entries()), [e.a for e in launches("newton_small_kernel")])
""".replace("N,", "%d," % n))
    assert out[:4] == ["1 [3]"] * 4, out
