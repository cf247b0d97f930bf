"""The library's host code over a stand-in HIP runtime (fake_hip.cpp): what
happens with several devices, when memory runs out, and when a call fails."""
import pytest

import fake_gpu


@pytest.fixture(scope="module")
def so(tmp_path_factory):
    lib = fake_gpu.build(str(tmp_path_factory.mktemp("fake")))
    if lib is None:
        pytest.skip("g++ not found")
    return lib


def test_calls_with_another_device_current(so):
    """Scratch and staging belong to the device of the lattice's stream, also
    where the calling thread's current device is another one."""
    out = fake_gpu.run(so, """
L = lbm.Lattice(700, 900, 0.7, 0.3, "f64")
P = lbm.Pool(1 << 30, "f32")
s = P.add(800, 900, 0.7, 0.3)
P.init(s, None, None, None)
P.step([s], 4)
assert fake.hipSetDevice(1) == 0
used = fake.fake_used(1)
fake.fake_log()
L.init(np.zeros((900, 700)), None, None)
L.step(3)
f = L.get_f()          # 45 MB: the staged copy
rho = L.moments()[0]   # 15 MB: the runtime's
P.init(s, None, None, None)
P.step([s], 4)
g = P.get_f(s)
assert not f.any() and not rho.any() and not g.any()  # no kernel ran: all memory is zero
assert "foreign" not in fake.fake_log().decode()
assert fake.fake_used(1) == used
import ctypes
d = ctypes.c_int(-1)
fake.hipGetDevice(ctypes.byref(d))
assert d.value == 1
print("ok")
""")
    assert out.strip() == "ok"
