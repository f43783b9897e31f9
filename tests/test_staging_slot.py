"""The wait for a staging slot (csrc/staging_slot.h), built for the host: each state goes where it should, a flag that is late
is waited for, and only an error ends a wait.  CPU only."""
import ctypes as C
import os
import subprocess
import threading
import time

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2504_14775_amd", "csrc")
SOURCE = r"""
#include "staging_slot.h"
extern "C" int await(int* state, uint32_t batch, const volatile uint32_t* flag, int (*settle)(), int (*error)()) {
    StagingSlot slot;
    slot.state = (StagingSlot::State)*state;
    slot.batch = batch;
    const int e = await_staging_slot(slot, flag, settle, error);
    *state = (int)slot.state;
    return e;
}
"""
FREE, COPIED, FLAGGED = 0, 1, 2
CALL = C.CFUNCTYPE(C.c_int)


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("staging_slot")
    (d / "slot.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O2", "-shared", "-fPIC", "-pthread", "-I", CSRC, str(d / "slot.cpp"), "-o", str(d / "slot.so")], check=True)
    lib = C.CDLL(str(d / "slot.so"))
    lib.await_ = getattr(lib, "await")
    lib.await_.argtypes = [C.POINTER(C.c_int), C.c_uint32, C.POINTER(C.c_uint32), CALL, CALL]
    return lib


def wait(lib, state, batch, flag, settle=0, errors=(), write=None, write_when_asked=None):
    """(result, state after, calls of settle, calls of error); write = (delay, number) stores a flag meanwhile, write_when_asked
    one when the second question for an error comes."""
    calls = {"settle": 0, "error": 0}

    def on_settle():
        calls["settle"] += 1
        return settle

    def on_error():
        calls["error"] += 1
        if write_when_asked is not None and calls["error"] == 2:
            word.value = write_when_asked
        return errors[min(calls["error"], len(errors)) - 1] if errors else 0

    st, word = C.c_int(state), C.c_uint32(flag)
    writer = None
    if write:
        writer = threading.Timer(write[0], lambda: setattr(word, "value", write[1]))
        writer.start()
    e = lib.await_(C.byref(st), batch, C.byref(word), CALL(on_settle), CALL(on_error))
    if writer:
        writer.join()
    return e, st.value, calls["settle"], calls["error"]


def test_a_free_slot_is_not_waited_for(lib):
    assert wait(lib, FREE, 7, 3) == (0, FREE, 0, 0)


@pytest.mark.parametrize("batch", [1, 7, 0, 2 ** 32 - 1])
def test_a_flag_with_the_number_of_the_batch_frees_the_slot(lib, batch):
    assert wait(lib, FLAGGED, batch, batch) == (0, FREE, 0, 0)


@pytest.mark.parametrize("delay", [0.0005, 0.05])
def test_an_older_number_is_waited_out(lib, delay):
    """Also where the wait is long enough to sleep between its looks."""
    t = time.monotonic()
    assert wait(lib, FLAGGED, 8, 7, write=(delay, 8)) == (0, FREE, 0, 0)
    assert time.monotonic() - t >= delay


def test_there_is_no_limit_of_time_and_no_error_means_on(lib):
    """Asked for an error twice, none there: the flag is waited for."""
    assert wait(lib, FLAGGED, 8, 7, write_when_asked=8) == (0, FREE, 0, 2)


def test_an_error_ends_the_wait_and_the_slot_stays_taken(lib):
    assert wait(lib, FLAGGED, 8, 7, errors=(0, 719)) == (719, FLAGGED, 0, 2)


def test_a_slot_without_a_flag_is_settled(lib):
    """Whatever an earlier batch left in its flag."""
    assert wait(lib, COPIED, 8, 8) == (0, FREE, 1, 0)
    assert wait(lib, COPIED, 8, 7) == (0, FREE, 1, 0)
    assert wait(lib, COPIED, 8, 7, settle=719) == (719, COPIED, 1, 0)
