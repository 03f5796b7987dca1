"""The bins and windows of the backward's record scatter, planned on the host."""
import ctypes as C
import math
import os
import re

import numpy as np
import pytest

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


def _plan(voxels, size):
    g, b = Grid(), Bins()
    for a in range(3):
        g.p0[a], g.p1[a] = 0.0, size[a]
    for l, v in enumerate(voxels):
        g.voxel[l] = v
        for a, f in enumerate((g.nx, g.ny, g.nz)):
            f[l] = max(2, math.ceil(round(size[a] / v, 6)) + 1)
    G.lib()._ZN2gs9plan_binsERKNS_4GridERNS_4BinsE(C.byref(g), C.byref(b))
    return b


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
