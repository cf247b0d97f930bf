"""Which kernels lbm_step launches, read off the library's own launches over
a stand-in HIP runtime (fake_hip.cpp)."""
import pytest

import fake_gpu

DEFAULT = {"f64": (1, 16, 16 | 32 | 2), "f32": (2, 16, 16 | 32 | 2), "f32s": (2, 16, 16 | 32 | 2), "f16s": (1, 32, 16 | 32)}


@pytest.fixture(scope="module")
def so(tmp_path_factory):
    lib = fake_gpu.build(str(tmp_path_factory.mktemp("fake")))
    if lib is None:
        pytest.skip("g++ not found")
    return lib


def case(nx, ny, dtype, *calls, **kw):
    return dict({"nx": nx, "ny": ny, "dtype": dtype, "calls": calls}, **kw)


@pytest.mark.parametrize("dtype", DEFAULT)
def test_a_shape_given_without_the_defaults_h_is_that_kernel_alone(so, dtype):
    """The default two-step shape as lbm_get_tile reports it takes block and
    cascade passes, as a new lattice does; with any other h it takes pairs
    only, so that the two-step kernel can be had (and tested) by itself."""
    vx, nw, flags = DEFAULT[dtype]
    sizes = [(64, 64), (4000, 4), (2400, 2400)]
    new, own, pairs, field = (
        [case(nx, ny, dtype, 9, **kw) for nx, ny in sizes]
        for kw in ({}, {"tile": "own"}, {"tile": (vx, nw, 0, flags)}, {"tile": (vx, nw, 0, flags), "field": True}))
    got = fake_gpu.routes(so, new + own + pairs + field)
    assert got[:3] == got[3:6]
    assert set(got[0]) == {"block", "step"} and set(got[1]) == {"block"}
    assert got[2][0] in ("cascade8", "cascade4")
    assert all(r == ["pair"] * 4 + ["step"] for r in got[6:])


def test_the_environments_shape_follows_the_same_rule(so):
    c = [case(64, 64, "f32", 8)]
    assert fake_gpu.routes(so, c, {"LBM_TILE": "2,16,0,50"}) == [["pair"] * 4]
    assert fake_gpu.routes(so, c, {"LBM_TILE": "2,16,8,50"}) == [["block"] * 2]


def test_the_cascade_sizes_take_cascade_passes(so):
    import cascade_sizes
    cases = list(cascade_sizes.cases())
    got = fake_gpu.routes(so, [case(nx, ny, dtype, steps, steps + 5, **kw) for dtype, steps, nx, ny, _, kw in cases])
    for (dtype, steps, nx, ny, name, _), r in zip(cases, got):
        r = [k for k in r if k != "ghosts"]  # FP16: after each call's passes
        tail = ["step"] + (["xbc"] if name == "inlet" else [])
        first = "cascade%d" % steps
        assert r[0] == first and r[1] == first, (dtype, steps, nx, ny, name, r)
        assert r[2:] == ["cascade4"] + tail, (dtype, steps, nx, ny, name, r)


def test_the_two_step_sizes_take_pairs(so):
    import cascade_sizes
    cases = list(cascade_sizes.pair_cases())
    got = fake_gpu.routes(so, [case(nx, ny, dtype, 7, **kw) for dtype, nx, ny, kw in cases])
    for c, r in zip(cases, got):
        assert r == ["pair"] * 3 + ["step"], (c, r)


def test_one_fp16_step_with_an_inlet_takes_the_faster_launches(so):
    """Where a single-step launch and one for the boundaries are faster than a block
    pass of one step (from 1500 tiles), a lone step takes them."""
    inlet = {"inlet": (0.01, 50.0)}
    got = fake_gpu.routes(so, [case(nx, ny, "f16s", n, **inlet)
                               for nx, ny in ((650, 650), (700, 700), (5000, 100)) for n in (1, 2)])
    assert got == [["block"], ["block"], ["step", "xbc"], ["block"], ["step", "xbc"], ["block"]]


@pytest.mark.parametrize("dtype", ["f64", "f32", "f32s"])
def test_the_pool_sizes_take_cascade_passes(so, dtype):
    import cascade_sizes
    out = fake_gpu.run(so, fake_gpu.PASSES + f"""
for mode in (lbm.GROUPED, lbm.GRAPH, lbm.PERSISTENT):
    P = lbm.Pool(1 << 34, {dtype!r})
    P.set_mode(mode)
    slots = [P.add(nx, ny, 0.7, 0.3) for nx, ny in {cascade_sizes.POOL_SHAPES!r}]
    for s in slots: P.init_device(s, None, None, None)
    fake.fake_log()
    for c in {cascade_sizes.POOL_COUNTS!r}:
        P.step(slots, np.array(c, dtype=np.int32))
        r = passes(fake.fake_log())
        # a replayed graph of the first call launches nothing by itself
        assert r.count("pool_cascade4") == (1 if mode == lbm.PERSISTENT else max(c) // 4) or (mode == lbm.GRAPH and not r), (mode, c, r)
        assert "pool_pair" in r or not any(n % 4 for n in c) or not r
print("ok")
""")
    assert out.strip() == "ok"
