"""Lattices whose steps the cascade kernel takes, by storage type and steps
per pass: strips of 112, 96 (eight steps) and 240 (FP16) columns, of which the
last holds 1 to 4 columns, one column less than all, or all; widths of every
remainder of a lane's columns; one strip alone; and lattices hardly higher than a
pass's halo. test_routes.py checks on the CPU that the passes are taken,
test_gpu_cascade_sizes.py on the GPU that they give the bits of single steps."""

SIZES = {
    ("f64", 4): [(111, 5405), (113, 10619), (225, 22222), (337, 1780), (338, 1775), (449, 1336), (450, 1333), (260003, 19)],
    ("f64", 8): [(95, 6315), (96, 6250), (225, 2666), (226, 2654), (561, 1069), (961, 2497), (962, 2494)],
    ("f32", 4): [(111, 5405), (112, 5357), (225, 2666), (226, 2654), (337, 1780), (338, 1775), (449, 1336), (260003, 19)],
    ("f32", 8): [(95, 52631), (96, 52083), (225, 10666), (226, 10619), (1921, 3643), (1922, 3642)],
    ("f32s", 4): [(111, 5405), (112, 5357), (225, 2666), (226, 2654), (337, 1780), (338, 1775), (449, 1336), (260003, 19)],
    ("f32s", 8): [(95, 52631), (96, 52083), (225, 10666), (226, 10619), (961, 5202), (962, 5197)],
    ("f16s", 4): [(237, 17721), (238, 17647), (239, 17573), (240, 17500), (483, 8695), (484, 8677), (721, 5825), (722, 5817),
                  (723, 5809), (724, 5801)],
}
INLET = (0.02, 17.0)
# what a lattice may have besides; a c2 field goes with four steps only
OPTIONS = {"plain": {}, "equilibrium": {"model": 1}, "inlet": {"inlet": INLET}, "field": {"field": True}}


def cases():
    for (dtype, steps), sizes in SIZES.items():
        for nx, ny in sizes:
            for name, kw in OPTIONS.items():
                if name != "field" or steps == 4:
                    yield dtype, steps, nx, ny, name, kw


# Between the sizes of the block and the cascade kernel: two-step passes
PAIR_SIZES = [(397, 391), (300, 277), (265, 333)]


def pair_cases():
    for dtype in ("f64", "f32", "f32s", "f16s"):
        for nx, ny in PAIR_SIZES + ([(1103, 1021)] if dtype == "f16s" else []):
            for name in ("plain", "equilibrium", "field"):
                yield dtype, nx, ny, OPTIONS[name]


# A batch whose calls take cascade passes: two lattices large enough to make them pay, and
# beside them narrow, low and ragged ones, whose strips wrap several times in x or y
POOL_SHAPES = [(1400, 1300), (1201, 1111), (3, 3), (4, 17), (5, 2003), (49, 503), (95, 78), (111, 305), (112, 170), (113, 301),
               (114, 97), (225, 61), (226, 9), (337, 14), (6001, 3), (700, 333)]
# steps of each call per slot: every remainder of four, below a pass, none
POOL_COUNTS = [(8, 13, 6, 7, 3, 0, 21, 4, 5, 9, 10, 11, 12, 14, 15, 16), (5, 4, 11, 1, 10, 16, 2, 9, 8, 7, 6, 4, 3, 13, 4, 0),
               (8, 13, 6, 7, 3, 0, 21, 4, 5, 9, 10, 11, 12, 14, 15, 16), (4,) * 16]
