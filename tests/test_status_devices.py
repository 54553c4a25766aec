"""pg_status_check with words that a kernel on the current device cannot read (another
device's, host memory): they are copied, as ever, and only the current device's own
words are read by a kernel.  On the host, with the runtime's calls stood in for."""
import pytest

from fake_hip import run

CODE = """
import numpy as np, synth
views = abi.pg_views_create([synth.pinhole(np.eye(3), np.zeros(3), 64, 48)], 1, 10, 0, abi.make_tiling())
over, count, need = C.c_int32({over}), C.c_int64((1 << 33) + 5), C.c_int64()
fake.fake_words{words}
st = lib.pg_status_check(C.addressof(over), C.addressof(count), C.byref(need), None)
assert st == ({over} and -3) and need.value == count.value, (st, need.value)
print(fake.fake_launches(), fake.fake_copies())
"""
DEVICE, HOST = 2, 1      # hipMemoryTypeDevice, hipMemoryTypeHost


@pytest.mark.parametrize("words,kernel", [((1, DEVICE, 0), True), ((1, DEVICE, 1), False), ((1, HOST, 0), False),
                                          ((0, 0, 0), False)],
                         ids=["current device", "another device", "pinned", "unknown"])
@pytest.mark.parametrize("over", [0, 1])
def test_only_the_current_devices_words_meet_a_kernel(tmp_path, words, kernel, over):
    launches, copies = map(int, run(tmp_path, CODE.format(over=over, words=words)).split())
    assert (launches, copies) == ((1, 0) if kernel else (0, 2))
