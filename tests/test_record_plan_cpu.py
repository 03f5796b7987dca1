"""The bins and windows of the backward's record scatter, planned on the host."""
import ctypes as C
import math
import os
import re

import numpy as np
import pytest

import synth
from paper_2206_14735_amd import gosurf as G

CSRC = os.path.join(os.path.dirname(os.path.abspath(G.__file__)), "csrc")


class Grid(C.Structure):
    _fields_ = [("p0", C.c_float * 3), ("p1", C.c_float * 3), ("voxel", C.c_float * 4), ("nx", C.c_int * 4),
                ("ny", C.c_int * 4), ("nz", C.c_int * 4), ("off", C.c_longlong * 4)]


class Bins(C.Structure):
    _fields_ = [("level", C.c_int), ("shift", C.c_int), ("nb", C.c_int * 3), ("last", C.c_int * 3),
                ("p0", C.c_float * 3), ("inv_v", C.c_float), ("wd", (C.c_int * 3) * 4), ("wbase", C.c_int * 4),
                ("ratio", C.c_float * 4)]


def _constant(name):
    src = open(os.path.join(CSRC, "bins.h")).read() + open(os.path.join(CSRC, "scatter.hip")).read()
    return int(re.search(rf"constexpr (?:int|unsigned) {name} = (\d+);", src).group(1))


def _bins(p0, p1, voxels, dims):
    g, b = Grid(), Bins()
    for a in range(3):
        g.p0[a], g.p1[a] = p0[a], p1[a]
    for l, v in enumerate(voxels):
        g.voxel[l] = v
        for a, f in enumerate((g.nx, g.ny, g.nz)):
            f[l] = dims[l][a]
    G.lib()._ZN2gs9plan_binsERKNS_4GridERNS_4BinsE(C.byref(g), C.byref(b))
    return b


def _plan(voxels, size):
    dims = [[max(2, math.ceil(round(s / v, 6)) + 1) for s in size] for v in voxels]
    return _bins([0.0] * 3, size, voxels, dims)


def records_from(layout, bf16=False, ragged=False):
    """Points (samples, and two per smoothness pair) from which a batch on this
    layout is scattered through records."""
    b = _bins(layout.p0, layout.p1, layout.voxels, layout.dims)
    kept = far = 0
    for d in layout.dims:   # levels the other way keeps on chip: coarsest first, 1024 vertices together
        n = d[0] * d[1] * d[2]
        if kept + n <= 1024:
            kept += n
        else:
            far += 1
    f = G.lib()._ZN2gs12records_fromERKNS_4BinsEibb
    f.restype = C.c_longlong
    return f(C.byref(b), far, C.c_bool(bf16), C.c_bool(ragged))


@pytest.mark.parametrize("thin", [0, 1, 2, None])
def test_windows_fit_the_lds_and_the_flush(thin):
    """Levels of any voxel ratio in boxes thin along one axis or none: the
    windows of a bin fit the LDS together, and no column along z is longer than
    a flush walks."""
    verts, edge = _constant("kWinVerts"), _constant("kWinEdge")
    rng = np.random.default_rng(0 if thin is None else 1 + thin)
    for _ in range(3000):
        fine = float(rng.uniform(0.02, 0.2))
        vox = [fine * float(rng.choice([1.0, rng.uniform(1.0, 1.2), rng.uniform(1.0, 4.0), rng.uniform(1.0, 32.0), 2.0, 4.0]))
               for _ in range(3)] + [fine]
        size = [fine * float(rng.uniform(16.0, 64.0)) for _ in range(3)]
        if thin is not None:
            size[thin] = fine * float(rng.uniform(1.0, 6.0))
        b = _plan(sorted(vox, reverse=True), size)
        assert sum(b.wd[l][0] * b.wd[l][1] * b.wd[l][2] for l in range(4)) <= verts
        assert max(b.wd[l][2] for l in range(4)) <= edge, (vox, size, b.shift)
        assert b.shift >= 2


# Backward times on MI355X, us: (voxels, box, samples, pairs, direct, through records)
ROOM, CUBE = ((0.0, 0.0, 0.0), (8.0, 6.0, 3.0)), ((-1.0,) * 3, (1.0,) * 3)
MEASURED = [
    ((0.03, 0.06, 0.24, 0.96), ROOM, 589824, 16384, 352, 388), ((0.03, 0.06, 0.24, 0.96), ROOM, 1248000, 0, 631, 662),
    ((0.03, 0.06, 0.24, 0.96), ROOM, 3145728, 16384, 1579, 1460), ((0.03, 0.06, 0.24, 0.96), ROOM, 6291456, 16384, 3050, 2701),
    ((0.02, 0.06, 0.24, 0.96), ROOM, 786432, 0, 423, 600), ((0.02, 0.06, 0.24, 0.96), ROOM, 1572864, 0, 807, 908),
    ((0.02, 0.06, 0.24, 0.96), ROOM, 3072000, 1 << 18, 1979, 1693), ((0.02, 0.06, 0.24, 0.96), ROOM, 4194304, 1 << 18, 2517, 2169),
    ((0.01, 0.06, 0.24, 0.96), ROOM, 3145728, 0, 1638, 2800), ((0.01, 0.06, 0.24, 0.96), ROOM, 6291456, 0, 3231, 4456),
    ((0.08, 0.16, 0.32, 0.64), CUBE, 32768, 0, 53, 68), ((0.08, 0.16, 0.32, 0.64), CUBE, 65536, 0, 72, 80),
    ((0.08, 0.16, 0.32, 0.64), CUBE, 65536, 4096, 91, 85), ((0.08, 0.16, 0.32, 0.64), CUBE, 131072, 0, 123, 100),
    ((0.05, 0.1, 0.2, 0.4), CUBE, 64000, 0, 74, 87), ((0.05, 0.1, 0.2, 0.4), CUBE, 128000, 0, 118, 103),
]


MEASURED_BF16 = [
    ((0.03, 0.06, 0.24, 0.96), ROOM, 393216, 0, 235, 238), ((0.03, 0.06, 0.24, 0.96), ROOM, 589824, 16384, 356, 306),
    ((0.03, 0.06, 0.24, 0.96), ROOM, 361968, 16384, 209, 216), ((0.03, 0.06, 0.24, 0.96), ROOM, 2097152, 16384, 1098, 746),
    ((0.02, 0.06, 0.24, 0.96), ROOM, 786432, 0, 429, 502), ((0.02, 0.06, 0.24, 0.96), ROOM, 1572864, 0, 822, 716),
    ((0.01, 0.06, 0.24, 0.96), ROOM, 6291456, 0, 3395, 3576),
    ((0.08, 0.16, 0.32, 0.64), CUBE, 32768, 0, 53, 65), ((0.08, 0.16, 0.32, 0.64), CUBE, 76800, 0, 81, 77),
    ((0.05, 0.1, 0.2, 0.4), CUBE, 64000, 0, 74, 84), ((0.05, 0.1, 0.2, 0.4), CUBE, 128000, 0, 119, 90),
]


@pytest.mark.parametrize("bf16,voxels,box,samples,pairs,direct,records",
                         [(False, *m) for m in MEASURED] + [(True, *m) for m in MEASURED_BF16])
def test_records_are_taken_where_they_were_faster(bf16, voxels, box, samples, pairs, direct, records):
    layout = synth.padded_layout(*box, voxels)
    assert (samples + 2 * pairs >= records_from(layout, bf16)) == (records < direct)
