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


def test_creation_takes_kept_scratch_back(so):
    """Scratch kept between calls is given back before an allocation is
    reported as failed: a lattice, a c2 field, a pool's slots, a larger scratch."""
    out = fake_gpu.run(so, """
MB = 1 << 20
L = lbm.Lattice(700, 900, 0.7, 0.3, "f64")
L.init(None, None, None)
big = lbm.Lattice(900, 1000, 0.7, 0.3, "f64")
big.init(None, None, None)

def tight(free):  # 45 MB of scratch kept, `free` left beside it
    fake.fake_limit(0, 1 << 40)
    L.get_f()
    fake.fake_limit(0, fake.fake_used(0) + free)

tight(10 * MB)
lbm.Lattice(500, 900, 0.7, 0.3, "f32").close()  # 34 MB
tight(1 * MB)
L.set_c2_field(np.full((900, 700), 0.3))  # the field itself takes 5 MB, its staging as much
fake.fake_limit(0, 1 << 40)
P = lbm.Pool(1 << 30, "f32")
tight(10 * MB)
P = lbm.Pool(40 * MB, "f32")
P.add(400, 900, 0.7, 0.3)  # the pool's chunk is its budget
tight(30 * MB)
big.get_f()  # 65 MB
for f, need in ((lambda: lbm.Lattice(2000, 2000, 0.7, 0.3, "f64"), 576 * MB),):  # what does not fit is still refused
    tight(10 * MB)
    try:
        f()
        raise SystemExit("accepted")
    except lbm.LBMError as e:
        assert e.status == lbm.ENOMEM
print("ok")
""")
    assert out.strip() == "ok"


def test_failed_read_leaves_no_copy_behind(so):
    """A read that fails half way has no copy under way into the caller's arrays."""
    out = fake_gpu.run(so, """
import ctypes
L = lbm.Lattice(70, 90, 0.7, 0.3, "f64")
L.init(None, None, None)
a, b = ctypes.c_void_p(), ctypes.c_void_p()
for p in (a, b):
    assert fake.hipHostMalloc(ctypes.byref(p), 70 * 90 * 8, 0) == 0
st = L._L.lbm_get_stream(L._h)
fake.fake_fail(b"hipMemcpyAsync", 1, fake_gpu.UNKNOWN)
assert L._L.lbm_moments(L._h, a, b, None, None) == lbm.EDEVICE
assert fake.fake_pending(st) == 0
assert L._L.lbm_moments(L._h, a, b, None, None) == lbm.OK
print("ok")
""")
    assert out.strip() == "ok"


@pytest.mark.parametrize("call,after", [("hipHostMalloc", 0), ("hipEventCreateWithFlags", 0),
                                        ("hipEventCreateWithFlags", 5)])
@pytest.mark.parametrize("error", [fake_gpu.OUT_OF_MEMORY, fake_gpu.CAPTURE_UNSUPPORTED])
def test_read_without_a_staging_ring(so, call, after, error):
    """Where no ring can be made (no pinned memory; another thread captures a
    graph) a large read goes as a small one does."""
    out = fake_gpu.run(so, f"""
L = lbm.Lattice(700, 900, 0.7, 0.3, "f64")
L.init(None, None, None)
fake.fake_fail(b"{call}", {after}, {error})
f = L.get_f()
assert not f.any()
assert fake.fake_pending(L._L.lbm_get_stream(L._h)) == 0
print("ok")
""")
    assert out.strip() == "ok"


def test_tuned_shapes_of_earlier_launches_are_timed_again(so, tmp_path):
    """A tune record whose key lacks the revision (written when the default
    shape stood for two-step launches) is not applied."""
    import json
    cache = tmp_path / "tune.jsonl"
    old = [("gfx950|lattice|1|1000x777", 4, 16, 8, 16), ("gfx950|pool|1|n2^1|s2^21", 4, 8, 2, 2)]
    cache.write_text("".join(json.dumps({"key": k, "vx": vx, "nw": nw, "h": h, "flags": f, "ch": 8, "us": 1.0}) + "\n"
                             for k, vx, nw, h, f in old))
    out = fake_gpu.run(so, """
fake.fake_fast(b"cascade_kernel")
with lbm.Lattice(1000, 777, 0.7, 0.3, "f32") as L:
    L.init_device(None, None, None)
    print(L.autotune(reps=1, use_cache=True) == L.get_tile() == (2, 16, 8, 50))
P = lbm.Pool(1 << 30, "f32")
s = [P.add(1000, 777, 0.7, 0.3) for _ in range(2)]
for k in s: P.init_device(k, None, None, None)
print(P.autotune(s, reps=1, use_cache=True) == (2, 16, 34))
""", {"LBM_TUNE_CACHE": str(cache)})
    assert out.split() == ["True", "True"]
    assert len(cache.read_text().splitlines()) == 4  # both were timed and recorded


def test_tuning_knows_the_boundaries(so):
    """A lattice with inlet/outlet boundaries is tuned on the launches it makes:
    the default's passes, against single steps and a boundary launch each, and not
    by a record of a periodic lattice."""
    out = fake_gpu.run(so, """
L = lbm.Lattice(350, 350, 0.7, 0.3, "f32")
L.init_device(None, None, None)
fake.fake_fast(b"step2_vstack_kernel<float, false, 1, 12")
print(L.autotune(reps=1, use_cache=True)[:2] == (1, 12))
L.set_x_boundaries(lbm.XBC_INLET_OUTLET, 1e-3, 500.0)
fake.fake_log()
fake.fake_fast(b"block_kernel")
print(L.autotune(reps=1, use_cache=True) == (2, 16, 8, 50))
log = fake.fake_log().decode()
print("xbc_kernel" in log and "step2_vstack" not in log)
L.set_x_boundaries(lbm.XBC_PERIODIC)
fake.fake_log()
print(L.autotune(reps=1, use_cache=True)[:2] == (1, 12) and not fake.fake_log())  # its own record
""")
    assert out.split() == ["True"] * 4
