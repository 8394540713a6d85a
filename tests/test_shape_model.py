"""The modelled tile shapes of multi-sweep passes over several grids (host-only)."""
import ctypes
import math
import random
import time

import pytest

from paper_2409_18824_amd import j3d

PLANES = (4, 6, 8, 10, 12, 16, 20, 24, 32, 48, 64)
# latency of a plane step, growing with the rows of a thread; per row on a CU; steps beyond the planes
COST = {(2, j3d.F32): (0.4, 0.056, 0.006, 3), (2, j3d.F64): (0.5, 0.047, 0.014, 6),
        (3, j3d.F32): (0.3, 0.0026, 0.01, 3), (3, j3d.F64): (0.3, 0.115, 0.042, 4)}


class Shape(ctypes.Structure):
    _fields_ = [(k, ctypes.c_int) for k in ("rows", "planes", "variant", "persistent", "order", "cols")]


def modelled_shape(sweeps, dtype, grids):
    fn = j3d._lib._ZN3j3d14modelled_shapeEiiPKNS_7ExtentsEi
    fn.restype = Shape
    n = len(grids)
    return fn(sweeps, dtype, (ctypes.c_int * (3 * n))(*[v for g in grids for v in g]), n)


def reference(sweeps, dtype, grids):
    """The estimate as it is stated, shape by shape and grid by grid."""
    f32 = dtype == j3d.F32
    lat, lat_row, row, fill = COST[sweeps, dtype]
    best, best_t = None, 1e300
    for rows in (2, 4, 8, 16):
        for ry in (2, 4):
            if not (4 if sweeps == 2 else 8) <= rows * ry <= 32 or (sweeps == 2 and rows == 16):
                continue
            out = rows * ry - 2 * (sweeps - 1)
            waves = (16 if ry == 2 or f32 else 12) if sweeps == 3 else (24 if ry == 2 or f32 else 16)
            cap = max(1, waves // rows)
            for planes in PLANES:
                tiles = sum(-(-nx // (64 - 2 * sweeps)) * -(-ny // out) * -(-nz // planes) for nx, ny, nz in grids)
                full, part = divmod(math.ceil(tiles / 256), cap)
                step = [lat + lat_row * ry + row * w * rows * ry for w in (cap, part)]
                t = (min(planes, max(g[2] for g in grids)) + fill) * (full * step[0] + (step[1] if part else 0.0))
                if t < best_t * (1.0 - 1e-12):
                    best, best_t = (rows, planes, 20 if ry == 4 else 6, 0, 0, 1), t
    return best


@pytest.mark.parametrize("sweeps", [2, 3])
@pytest.mark.parametrize("dtype", [j3d.F64, j3d.F32])
def test_shapes_are_those_of_the_estimate(sweeps, dtype):
    rng = random.Random(17)
    for n in (1, 1, 1, 2, 7, 64, 65, 256):
        for hi in (8, 64, 300, 4000):
            grids = [tuple(rng.randint(1, hi) for _ in range(3)) for _ in range(n)]
            s = modelled_shape(sweeps, dtype, grids)
            assert tuple(getattr(s, k) for k, _ in Shape._fields_) == reference(sweeps, dtype, grids), (n, hi)


def test_the_estimate_does_not_cost_a_cycle():
    """A server estimates shapes for up to 256 grids between two cycles, while
    the GPU waits: at most a quarter of what 256 estimates of one grid take (the
    tiles of all shapes counted in one walk; a third of it before)."""
    rng = random.Random(18)
    grids = [tuple(rng.randint(12, 48) for _ in range(3)) for _ in range(256)]

    def best(fn):
        ts = []
        for _ in range(15):
            t = time.perf_counter()
            fn()
            ts.append(time.perf_counter() - t)
        return min(ts)

    fn = j3d._lib._ZN3j3d14modelled_shapeEiiPKNS_7ExtentsEi
    fn.restype = Shape
    a = (ctypes.c_int * 768)(*[v for g in grids for v in g])
    together = best(lambda: fn(3, j3d.F64, a, 256))
    alone = best(lambda: [fn(3, j3d.F64, a, 1) for _ in range(256)])
    assert together < 0.25 * alone, (together, alone)
