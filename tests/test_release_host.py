"""Host build of the releases of slots (give_back_slots and release_beside in
csrc/smmo_device.hpp): blocks re-activated, emptied and freed, the switches
passed on over one to three levels of bitmaps.  Compiled for the host with a
stand-in for HIP (a wavefront of one lane); no GPU."""

from test_search_host import run


def test_releases_leave_the_states_of_the_model(tmp_path):
    assert run(tmp_path, "release_host") == {"wrong": 0, "errors": 0}
