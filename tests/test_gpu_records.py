"""The backward's scatter through records and per-bin windows against the oracle."""
import dataclasses

import numpy as np
import pytest

import synth
from tests.helpers import f32_layout, sphere_case
from tests.test_gpu_parity import _clear, compare, oracle_pair, run_device

pytestmark = pytest.mark.gpu


def _thin_case(voxels, size, M, S=777):
    """Rays along z through a box thin in x."""
    lo, hi = tuple(-s / 2 for s in size), tuple(s / 2 for s in size)
    dims = [tuple(int(np.ceil(round(s / v, 6))) + 1 for s in size) for v in voxels]
    L = f32_layout(synth.GridLayout(lo, hi, list(voxels), dims))
    grid, mlp = synth.init_params(L, seed=5, grid_std=0.3)
    _, _, b, _, _ = sphere_case(M=M, S=S)
    rng = np.random.default_rng(3)
    u = lambda n, k: rng.uniform(-1.0, 1.0, (n, k))  # noqa: E731
    half = np.array(size) / 2
    o = np.stack([0.9 * half[0] * u(M, 1)[:, 0], 0.9 * half[1] * u(M, 1)[:, 0], np.full(M, lo[2] - 0.15)], 1)
    r = np.concatenate([u(M, 2) * [0.01, 0.2], np.ones((M, 1))], 1)
    b = dataclasses.replace(b, o=o.astype(np.float32), r=r.astype(np.float32),
                            xs=(0.98 * half * u(len(b.xs), 3)).astype(np.float32))
    return L, _clear(grid, mlp, L, b), grid, mlp


@pytest.mark.parametrize("M", [200, 1250])
@pytest.mark.parametrize("voxels,size", [((0.64, 0.32, 0.083, 0.08), (0.24, 2.56, 2.56)),
                                         ((0.7, 0.3, 0.077, 0.07), (0.2, 2.1, 2.1))])
def test_close_levels_in_a_thin_box(voxels, size, M):
    """A bin of 8^3 cells touches up to ten vertices per axis of a level whose
    voxel is a little larger than the finest, and a thin box leaves room for such
    a window; such grids take bins of 4^3 cells.  Both batches are dense enough
    for records at 8^3 cells, the larger one at 4^3 as well."""
    L, b, grid, mlp = _thin_case(voxels, size, M)
    assert 7 < 8 * voxels[3] / voxels[2] < 8
    for shift in (3, 2)[:1 if M == 200 else 2]:
        bins = int(np.prod([((n - 2) >> shift) + 1 for n in L.dims[3]]))
        assert bins <= 256 and len(b.t) + 2 * len(b.xs) >= (512 if M == 200 else 1024) * bins
    compare(run_device(L, b, grid, mlp), *oracle_pair(grid, mlp, L, b), case=(L, b, mlp))
