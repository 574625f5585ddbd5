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
