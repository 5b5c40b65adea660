"""Grids a cell or two thick: the tiles that the thermal assembly and the
gradient take on them, and the gradient's of 8 x 4 x 2 cells, at their edges,
against the oracle, and a launch of more than 2^32 threads."""
import pytest
import torch

import test_gpu_grad_tiles as tg
import test_gpu_thermal as tt
from paper_1812_03952_amd import rsolve as rs

pytestmark = pytest.mark.gpu

COLUMNS = [(64, 1, 1), (65, 1, 1), (1, 64, 1), (1, 129, 1), (1, 1, 63), (1, 1, 130)]
PLANES = [(1, 8, 8), (1, 9, 17), (1, 23, 2), (1, 2, 70), (2, 1, 65), (5, 9, 1)]


@pytest.mark.parametrize("dims", COLUMNS + PLANES)
def test_thermal_matches_oracle(dims):
    tt.test_assembly_matches_oracle(dims)


GRAD = [(64, 1, 1), (65, 1, 1), (1, 64, 1), (1, 131, 1), (1, 1, 65), (1, 8, 8), (1, 9, 17), (8, 1, 8), (9, 1, 17),
        (8, 4, 2), (9, 5, 3), (24, 8, 5)]


@pytest.mark.parametrize("dims", GRAD)
def test_gradient_matches_oracle(dims):
    tg.test_assembly_and_gradient_tiles(dims)


def test_thermal_past_2_32_threads():
    """2 x 1 x 34 million cells, the states repeating every 1000 layers: the
    residual of the inner layers repeats as on a small grid, to the end."""
    period, reps = 1000, 34000
    tp = tt._tp((2, 1, 3 * period))
    q = rs.thermal_params()
    d, u, u0 = tt._device(tp, q)
    none = dict(wcell=torch.empty(0, dtype=torch.int32, device="cuda"), wkind=torch.empty(0, dtype=torch.int32, device="cuda"),
                wval=torch.empty(0, dtype=torch.float64, device="cuda"))

    def residual(nz, inputs):
        res = torch.full((8 * nz,), float("nan"), dtype=torch.float64, device="cuda")
        rs.thermal_assemble(2, 1, nz, q, inputs["kx"], inputs["ky"], inputs["kz"], inputs["u"], inputs["u0"],
                            none["wcell"], none["wkind"], none["wval"], None, res)
        return res

    one = dict(kx=d["kx"], ky=d["ky"], kz=d["kz"], u=u, u0=u0)
    one = {k: v[: v.numel() // 3].contiguous() for k, v in one.items()}
    small = residual(3 * period, {k: v.repeat(3) for k, v in one.items()}).view(3, -1)
    big = residual(reps * period, {k: v.repeat(reps) for k, v in one.items()}).view(reps, -1)
    assert torch.equal(big[0], small[0]) and torch.equal(big[-1], small[2])
    assert (big[1:-1] == small[1]).all()
    rs.pool_trim()

