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


@pytest.mark.parametrize("call", ["energy_grad", "energy", "noalloc"])
def test_evaluations_under_capture_before_the_sectors_tables(run, call):
    # under hubbard_set_timing the full vector's plan is uploaded and no sector
    # table; a capture after that launches what is there and allocates nothing,
    # and the next eager call runs on the sector
    run(f"""
for kw in (dict(), dict(V_bond=[0.5] * 7)):
    m = Model(1, 8, 2, U=4.0, **kw)
    m.timing(True)
    assert m.energy_grad()[0] == 0 and m.energy()[0] == 0
    m.timing(False)
    hh.hh_capture(1)
    st, k = m.{call}()
    assert st == 0 and has(k, "6k_pass") and not has(k, "k_sec"), (st, k)
    assert hh.hh_refused_in_capture() == 0 and hh.hh_last_error() == 0
    hh.hh_capture(0)
    assert m.energy_grad()[0] == 0
    st, k = m.{call}()
    assert st == 0 and has(k, "k_sec") and not has(k, "6k_pass"), (st, k)
    hh.hh_capture(1)            # the tables are there now
    assert m.{call}() == (0, k) and hh.hh_refused_in_capture() == 0
    hh.hh_capture(0)
""")


def test_h_and_states_under_capture_before_their_tables(run):
    run("""
m = Model(1, 8, 2, U=4.0, V_bond=[0.5] * 7)
m.timing(True)
assert m.apply_h()[0] == 0 and m.ansatz()[0] == 0
m.timing(False)
hh.hh_capture(1)
st, k = m.apply_h()
assert st == 0 and has(k, "6k_pass") and not has(k, "gather"), (st, k)
st, k = m.prepare()             # by init and the pass kernels
assert st == 0 and has(k, "6k_pass") and not has(k, "k_sec"), (st, k)
assert hh.hh_refused_in_capture() == 0
hh.hh_capture(0)
st, k = m.apply_h()
assert st == 0 and has(k, "gather") and not has(k, "6k_pass"), (st, k)
st, k = m.prepare()
assert st == 0 and has(k, "k_sec_expand"), (st, k)
hh.hh_capture(1)
assert has(m.apply_h()[1], "gather") and has(m.prepare()[1], "k_sec_expand")
assert hh.hh_refused_in_capture() == 0
""")


def test_calls_that_others_prepared_can_still_be_captured(run):
    # a prepared state uploads ansatz_apply's plan, a batch its members'
    # energy_grad plans: the calls that use them need no first call of their own
    run("""
m = Model(1, 8, 2, U=4.0)
assert m.prepare()[0] == 0
hh.hh_capture(1)
st, k = m.ansatz()
assert st == 0 and has(k, "6k_pass") and hh.hh_refused_in_capture() == 0, (st, k)
hh.hh_capture(0)
a, b = Model(1, 6, 2, U=4.0), Model(2, 2, 2, U=2.0, V_bond=[0.5] * 4)
for m in (a, b):
    m.work(abi.HUBBARD_OP_ENERGY_GRAD)
st, k = Batch([a, b]).energy_grad()
assert st == 0 and has(k, "k_sec_whole_batch"), (st, k)
hh.hh_capture(1)
for m in (a, b):
    st, k = m.energy_grad()
    assert st == 0 and has(k, "k_sec_whole"), (st, k)
    assert m.noalloc() == (st, k)
assert hh.hh_refused_in_capture() == 0
""")


def test_a_circuit_that_the_plan_refuses_is_refused(run):
    # 400 layers of a 2x2 cluster in one tile need more LDS than there is
    run("""
m = Model(2, 2, 400, U=4.0)
assert m.ansatz() == (abi.HUBBARD_ERR_ARG, [])
assert m.prepare() == (abi.HUBBARD_ERR_ARG, [])
assert b"more LDS" in L.hubbard_last_error()
""")


# the ways in which the sector's tables cannot be had: no device memory for the
# first allocation of them, and none on the host (any block of 1 KiB or more)
NO_MEMORY = {"device": ("hh.hh_fail_next(1)", "hh.hh_fail_next(0)"),
             "host": ("hh.hh_throw_above(1024)", "hh.hh_throw_above(0)")}


@pytest.mark.parametrize("where", list(NO_MEMORY))
@pytest.mark.parametrize("call", ["energy_grad", "energy"])
def test_full_vector_where_the_sectors_tables_do_not_fit(run, call, where):
    # with the full vector's plan there: the call runs it, reports nothing and
    # leaves no error behind; once there is memory the sector is used
    begin, end = NO_MEMORY[where]
    run(f"""
m = Model(2, 6, 2, U=4.0)
m.timing(True)
assert m.energy_grad()[0] == 0 and m.energy()[0] == 0
m.timing(False)
before = L.hubbard_last_error()
{begin}
st, k = m.{call}()
{end}
assert st == 0 and has(k, "6k_pass") and not has(k, "k_sec"), (st, k, L.hubbard_last_error())
assert hh.hh_last_error() == 0 and L.hubbard_last_error() == before
st, k = m.{call}()
assert st == 0 and has(k, "k_sec"), (st, k)
""")


@pytest.mark.parametrize("where", list(NO_MEMORY))
def test_state_and_batch_where_the_sectors_tables_do_not_fit(run, where):
    begin, end = NO_MEMORY[where]
    run(f"""
m = Model(2, 6, 2, U=4.0)
m.ansatz()
{begin}
st, k = m.prepare()
{end}
assert st == 0 and has(k, "6k_pass") and not has(k, "k_sec"), (st, k)
assert hh.hh_last_error() == 0
assert has(m.prepare()[1], "k_sec_expand")
if {where!r} == "device":
    # a batch whose members' plans are there: the sector's tables come first, then
    # (the second time) the batch's own
    for fail in (1, 2):
        ms = [Model(1, 6, 2, U=4.0), Model(1, 8, 2, U=4.0)]
        b = Batch(ms)
        for x in ms:
            x.timing(True)
            assert x.energy_grad()[0] == 0
            x.timing(False)
        if fail == 2:
            for x in ms:
                assert x.energy_grad()[0] == 0
        {begin}
        st, k = b.energy_grad()
        assert st == 0 and has(k, "k_batch_pass") and not has(k, "k_sec"), (st, k)
        assert hh.hh_last_error() == 0
""")


def test_sector_calls_report_what_does_not_fit(run):
    # the sector's own entry points have no other route: a status, no exception
    run("""
m = Model(2, 4, 2, U=4.0)
n = ctypes.c_size_t()
size = lambda: L.hubbard_sector_workspace_size(m.h, 2, abi.HUBBARD_SECTOR_ENERGY_GRAD,
                                               ctypes.byref(n))
hh.hh_fail_next(1)
assert size() == abi.HUBBARD_ERR_DEVICE and hh.hh_last_error() == 0
hh.hh_throw_above(1024)
st = size()
hh.hh_throw_above(0)
assert st == abi.HUBBARD_ERR_NOMEM
assert size() == 0 and m.sector_eg()[0] == 0
""")


def test_batch_takes_the_workspace_that_the_full_vectors_need(run):
    # many tiny instances need more bytes on their sectors than on the full
    # vectors; a caller's buffer of the latter size is taken, and used so
    run("""
ms = [Model(1, 2, 3, U=4.0) for _ in range(64)]
b = Batch(ms)
# one more member without layers keeps the batch on the full vectors: 64 members'
# need is less than that of 65, and the sectors' more
full = Batch(ms + [Model(1, 2, 0, U=4.0)]).need
assert full < b.need
st, k = b.energy_grad(full)
assert st == 0 and has(k, "k_batch_pass") and not has(k, "k_sec"), (st, k)
st, k = b.energy_grad()
assert st == 0 and has(k, "k_sec_whole_batch"), (st, k)
st, k = b.energy_grad(full)        # the same buffers, the smaller size again
assert st == 0 and has(k, "k_batch_pass"), (st, k)
assert b.energy_grad(512 * 64 - 1)[0] == abi.HUBBARD_ERR_SIZE
""")


def test_batch_builds_the_start_state_of_a_member_without_layers(run):
    # it has no forward pass that would; H's pass reads the state
    run("""
ms = [Model(1, 4, 2, U=4.0), Model(1, 4, 0, U=4.0), Model(2, 2, 0, U=4.0)]
for timed in (False, True):
    ms[0].timing(timed)
    b = Batch(ms)
    for _ in range(2):
        st, k = b.energy_grad()
        assert st == 0 and sum("k_init_basis" in x for x in k) == 2, (st, k)
        assert k.index([x for x in k if "k_batch_pass" in x][0]) == 2
""")
