"""The host side of the calls that run on the start state's sector, against the
stand-in runtime of host_hip.py: which kernels a call launches, and what
it does where it cannot allocate."""
import pytest

import host_hip


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    lib = host_hip.build(str(tmp_path_factory.mktemp("hip")))
    return lambda program: host_hip.run(lib, program)


def test_one_handles_planning_does_not_stop_another(run):
    # the first call of a new handle waits in its upload; a call on another
    # handle goes on
    run("""
import threading, time
ready, new = Model(2, 2, 2, U=4.0), Model(1, 6, 2, U=4.0)
assert ready.energy_grad()[0] == 0
hh.hh_hold(1)
st = []
t = threading.Thread(target=lambda: st.append(new.sector_eg()[0]))
t.start()
end = time.time() + 15
while not hh.hh_held() and time.time() < end:
    time.sleep(0.01)
assert hh.hh_held() == 1
assert ready.energy_grad()[0] == 0 and ready.noalloc()[0] == 0
assert hh.hh_held() == 1      # not after the other's upload had ended
hh.hh_hold(0)
t.join()
assert st == [0]
""")
